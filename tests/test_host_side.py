"""librasp's host-side headers, compiled for the CPU against a model of the HIP
runtime (tests/hip_model)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, main):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(main)
    subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-pthread", "-I" + os.path.join(ROOT, "tests", "hip_model"),
                    "-I" + os.path.join(ROOT, "paper_2604_12902_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-2000:])


def test_whole_shape_of_every_memory_size(tmp_path):
    """k_whole's launch over all sizes a load accepts (1 to 2^30 words), those
    whose bytes of a wave's slots are a multiple of 2^32 among them: blocks that
    fit a compute unit's LDS, or none."""
    _run(tmp_path, r"""
#include "rasp_internal.h"
#include <cstdio>
#include <initializer_list>
#include <cstdlib>
using namespace rasp;
static void check(uint32_t n, uint64_t total, uint64_t lds, uint32_t cus)
{
    const WholeShape w = whole_shape(n, total, lds, cus);
    bool ok = n > kWholeMaxN ? w.blocks == 0 : w.slab == whole_lds_bytes(n, w.sh) && w.sh >= 2 && w.sh <= 6;
    if (w.blocks) ok = ok && uint64_t(kWholeWpb) * w.slab <= lds && w.blocks <= 8 * cus && (w.blocks - 1) * uint64_t(kWholeWpb) < total;
    if (n <= kWholeMaxN && lds == 160 * 1024) ok = ok && w.blocks;
    if (!ok) { std::printf("n %u total %llu lds %llu cus %u: sh %u slab %u blocks %u\n", n, (unsigned long long)total,
                           (unsigned long long)lds, cus, w.sh, w.slab, w.blocks); std::exit(1); }
}
int main()
{
    for (uint64_t lds : {64ull * 1024, 160ull * 1024})
        for (uint32_t cus : {1u, 32u, 256u})
            for (uint64_t total : {1ull, 5ull, 100003ull, (1ull << 32) - 1}) {
                for (uint32_t n = 1; n <= 4096; ++n) check(n, total, lds, cus);
                for (uint32_t k = 12; k <= 30; ++k)
                    for (uint32_t m = 1; (uint64_t(m) << k) <= kMaxMemWords && m <= 3; ++m)
                        for (int d = -3; d <= 0; ++d) check((m << k) + d, total, lds, cus);
            }
}
""")


HOSTCOPY = r"""
#include "rasp_hostcopy.h"
#include <cstdio>
#include <cstdlib>
using namespace rasp;
typedef std::vector<char> Bytes;
static Bytes noise(size_t n, unsigned seed)
{
    Bytes b(n);
    for (auto &c : b) c = char((seed = seed * 1664525u + 1013904223u) >> 24);
    return b;
}
static void expect(bool ok, const char *what) { if (!ok) { std::printf("%s\n", what); std::exit(1); } }
"""


def test_copies_of_a_call_that_failed_do_not_land_in_the_next_ones(tmp_path):
    """A fetch that gives up between its copies (no room for the next one), then
    a load: the fetch's copies, still in flight, may not land in the pinned area
    once the load has put its own bytes there."""
    _run(tmp_path, HOSTCOPY + r"""
int main()
{
    HostCopy h;
    Stream s;
    for (size_t n : {100u, 4096u, 262144u}) {
        const Bytes old = noise(n, 1), fresh = noise(n, 2);
        Bytes out(n), dev(n);
        h.begin();
        expect(h.get(0, out.data(), old.data(), n, &s) == hipSuccess, "get");
        h.begin();                       // the next call: the fetch never waited
        expect(h.put(0, dev.data(), fresh.data(), n, &s) == hipSuccess, "put");
        expect(hipStreamSynchronize(&s) == hipSuccess, "wait");
        expect(dev == fresh, "the load's bytes were overwritten");
        expect(h.flush(&s) == hipSuccess, "flush");
        // and one that waits delivers what it got
        h.begin();
        expect(h.get(0, out.data(), old.data(), n, &s) == hipSuccess && h.flush(&s) == hipSuccess && out == old, "fetch");
    }
}
""")


def test_copies_of_every_size(tmp_path):
    """Copies of every size, many of them in one call among them, move the right
    bytes in any order; the first 512 KiB of small ones need the area and nothing
    else, more and larger ones the chunks, events and helpers, and all of it is
    given back."""
    _run(tmp_path, HOSTCOPY + r"""
#include <dirent.h>
static int threads()
{
    int n = 0;
    DIR *d = opendir("/proc/self/task");
    while (dirent *e = readdir(d)) n += e->d_name[0] != '.';
    closedir(d);
    return n;
}
constexpr size_t MiB = 1 << 20;
int main()
{
    Stream s;
    const size_t most = 40 * MiB;
    const Bytes src = noise(most, 3);
    Bytes dev(most), out(most);
    auto wait = [&](HostCopy &h) { expect(hipStreamSynchronize(&s) == hipSuccess, "wait"); h.settled(); };
    auto up = [&](HostCopy &h, size_t n, size_t from = 0) {
        std::fill(dev.begin(), dev.begin() + n, 0);
        h.begin();
        expect(h.put(0, dev.data(), src.data() + from, n, &s) == hipSuccess, "put");
        wait(h);
        expect(std::equal(dev.begin(), dev.begin() + n, src.begin() + from), "up");
    };
    auto down = [&](HostCopy &h, size_t n) {
        std::fill(out.begin(), out.begin() + n, 0);
        h.begin();
        expect(h.get(0, out.data(), dev.data(), n, &s) == hipSuccess && h.flush(&s) == hipSuccess &&
               std::equal(out.begin(), out.begin() + n, dev.begin()), "down");
    };
    auto opened = [&](bool area, bool chunks) {
        const size_t want = (area ? HostCopy::kArea : 0) + (chunks ? HostCopy::kWorkers * HostCopy::kSlots * HostCopy::kChunk : 0);
        const bool ok = model().pinned_bytes == want && model().events == (chunks ? int(HostCopy::kWorkers * HostCopy::kSlots) : 0) &&
                        threads() == (chunks ? int(HostCopy::kWorkers) : 1);
        if (!ok) std::printf("area %d chunks %d: %zu bytes, %d events, %d threads\n", area, chunks, model().pinned_bytes,
                             model().events, threads());
        expect(ok, "opened");
    };
    {
        HostCopy h;
        for (size_t n : {1u, 300u, 4097u, 100000u}) {
            up(h, n, n % 7);
            down(h, n);
        }
        up(h, HostCopy::kOpenAfter - 2 * 104398);          // as much as does not open the chunks
        opened(true, false);
        up(h, 1);
        opened(true, true);
        for (size_t n : {262145u, 1048575u, 1048576u}) {
            up(h, n, n % 7);
            down(h, n);
        }
    }
    opened(false, false);
    {
        // many copies in one call, with waits within
        HostCopy h;
        std::fill(dev.begin(), dev.end(), 0);
        h.begin();
        size_t at = 0;
        for (int k = 0; k < 300; ++k) {
            const size_t n = size_t(k) * 3700 % 200003 + 1;
            expect(h.put(0, dev.data() + at, src.data() + at, n, &s) == hipSuccess, "put");
            at += n;
        }
        wait(h);
        expect(std::equal(dev.begin(), dev.begin() + at, src.begin()), "many up");
        h.begin();
        for (size_t x = 0, k = 0; x < at; ++k) {
            const size_t n = std::min(at - x, (k * 7919) % (k % 3 ? 5003 : 300007) + 1);
            expect(h.get(0, out.data() + x, dev.data() + x, n, &s) == hipSuccess, "get");
            x += n;
        }
        expect(h.flush(&s) == hipSuccess && std::equal(out.begin(), out.begin() + at, src.begin()), "many down");
    }
    opened(false, false);
    {
        HostCopy h;
        for (size_t n : {1048577u, 2097152u, 9000001u, 33554433u}) {
            up(h, n, 11);
            down(h, n);
        }
        opened(false, true);
        // copies in chunks and small ones in one call
        std::fill(dev.begin(), dev.end(), 0);
        h.begin();
        for (size_t at = 0, k = 0; at < most; ++k) {
            const size_t n = std::min(most - at, k % 2 ? size_t(4097) : 3 * MiB + k);
            expect(h.put(0, dev.data() + at, src.data() + at, n, &s) == hipSuccess, "put");
            at += n;
        }
        wait(h);
        expect(dev == src, "mixed up");
        std::fill(out.begin(), out.end(), 0);
        h.begin();
        for (size_t at = 0, k = 0; at < most; ++k) {
            const size_t n = std::min(most - at, k % 2 ? size_t(4097) : 3 * MiB + k);
            expect(h.get(0, out.data() + at, dev.data() + at, n, &s) == hipSuccess, "get");
            at += n;
        }
        expect(h.flush(&s) == hipSuccess && out == src, "mixed down");
        opened(true, true);
    }
    opened(false, false);
    {
        // pinned memory of the caller's own, and none to be had for the copies
        HostCopy h;
        void *p = nullptr;
        expect(hipHostMalloc(&p, 20 * MiB, 0) == hipSuccess, "pinned");
        memcpy(p, src.data(), 20 * MiB);
        std::fill(dev.begin(), dev.end(), 0);
        h.begin();
        expect(h.put(0, dev.data(), p, 20 * MiB, &s) == hipSuccess, "put");
        wait(h);
        expect(std::equal(dev.begin(), dev.begin() + 20 * MiB, src.begin()), "from pinned memory");
        hipHostFree(p);
        model().refuse = true;
        up(h, 5);
        up(h, 20 * MiB);
        down(h, 20 * MiB);
        down(h, 6);
        model().refuse = false;
        opened(false, false);
    }
    opened(false, false);
}
""")


def test_waves_of_a_work_list_are_spread_evenly():
    """A model of which waves of a launch over a list with memories in HBM look for
    machines: as many as find one (or all there are), and over compute units that
    take blocks in turn, and over the places of a block's waves, as evenly as
    whole blocks allow."""
    import numpy as np
    for cus in (1, 8, 64, 256):
        for wpb in (1, 2, 4):
            for per_cu in (1, 2, 4, 8):
                grid = cus * per_cu
                b, w = np.meshgrid(np.arange(grid), np.arange(wpb), indexing="ij")
                for need in sorted({0, 1, 2, 3, cus, cus + 1, cus * wpb - 1, cus * wpb, cus * wpb + 1, 3 * cus + 7,
                                    grid * wpb // 2, grid * wpb - 1, grid * wpb, grid * wpb + 9}):
                    used = min(grid, -(-need // (cus * wpb)) * cus)
                    on = (b < used) & (((w + b // cus) % wpb) * used + b < need)
                    assert on.sum() == min(need, grid * wpb), (cus, wpb, per_cu, need)
                    by_cu = np.bincount((b % cus)[on], minlength=cus)
                    blocks = max(1, used // cus)
                    assert by_cu.max() - by_cu.min() <= (blocks if need < used * wpb else 0), (cus, wpb, per_cu, need)
