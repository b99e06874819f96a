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


def test_small_copies_open_no_more_than_the_area(tmp_path):
    """Copies up to 256 KiB need the 1 MiB area and nothing else, larger ones
    the chunks, events and helpers only from the sizes and the sum that pay for
    them; every way moves the right bytes, and all of it is given back."""
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
int main()
{
    Stream s;
    const size_t most = 64 << 20;
    const Bytes src = noise(most, 3);
    Bytes dev(most), warm(most);
    auto up = [&](HostCopy &h, size_t n) {
        std::fill(dev.begin(), dev.begin() + n, 0);
        expect(h.begin() == hipSuccess && h.put(0, dev.data(), src.data(), n, &s) == hipSuccess &&
               hipStreamSynchronize(&s) == hipSuccess && std::equal(src.begin(), src.begin() + n, dev.begin()), "up");
        h.settled();
    };
    auto down = [&](HostCopy &h, char *out, size_t n) {
        expect(h.begin() == hipSuccess && h.get(0, out, dev.data(), n, &s) == hipSuccess && h.flush(&s) == hipSuccess &&
               std::equal(out, out + n, dev.begin()), "down");
    };
    auto down_new = [&](HostCopy &h, size_t n) {
        char *p = static_cast<char *>(mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
        down(h, p, n);
        munmap(p, n);
    };
    auto opened = [&](bool area, bool chunks) {
        expect(model().pinned_bytes == (area ? HostCopy::kArea : 0) + (chunks ? HostCopy::kWorkers * HostCopy::kSlots * HostCopy::kChunk : 0) &&
               model().events == (chunks ? int(HostCopy::kWorkers * HostCopy::kSlots) : 0) &&
               threads() == (chunks ? int(HostCopy::kWorkers) : 1), "opened");
    };
    {
        HostCopy h;
        for (size_t n : {1u, 300u, 262144u, 262145u, 1048575u}) {
            up(h, n);
            down(h, warm.data(), n);
            down_new(h, n);
            opened(true, false);
        }
    }
    opened(false, false);
    {
        HostCopy h;
        up(h, most - 1);                           // uploads below 64 MiB, downloads into pages that are there below 4
        for (int k = 0; k < 5; ++k) down(h, warm.data(), (4 << 20) - 1);
        for (int k = 0; k < 7; ++k) down_new(h, 1 << 20);    // 7 MiB of those that gain
        opened(false, false);
        down_new(h, 1 << 20);
        opened(false, true);
        for (size_t n : {1048576u, 1048577u, 2097152u, 4194304u, 9000001u}) {
            down(h, warm.data(), n);
            down_new(h, n);
        }
        opened(false, true);
    }
    opened(false, false);
    {
        HostCopy h;
        up(h, most);
        opened(false, true);
    }
    opened(false, false);
}
""")
