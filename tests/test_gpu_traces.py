"""GPU parity of the trace kernel and of the lists it hands on, bit-exact.

A persistent run with a first pass and a large enough budget compiles its
survivors into nodes (k_trace), steps the rest whole in LDS (k_whole) or on the
work queue.  Every field of every machine is compared with the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_2604_12902_amd import workloads as W
from test_gpu_parity import _boundary_programs, _image, _random_states, compare

pytestmark = pytest.mark.gpu


def _uniform(seed, num_vms, isa, n, w=32, m=12):
    """Random programs of 2m words over opcodes 1..8 with operands near the
    program, one n for all machines, two inputs and two outputs at most."""
    rng = np.random.Generator(np.random.PCG64(seed))
    words = rng.integers(-2, min(2 * m + 4, n + 3), (num_vms, 2 * m))
    words[:, ::2] = rng.integers(1, 9, (num_vms, m))
    words = words[:, :n]
    b = W.from_programs(isa, [list(map(int, r)) for r in words], n, [[3, -4]] * num_vms, ell=2, s=2)
    b.word_bits = w
    return b


def _wanderers(num_vms, n):
    """Counted stores through a moving address that ends up in the program:
    addresses new on every round, which no node holds."""
    LOAD, ADD, STORE, JMP = 1, 2, 4, 8
    progs = [_image(n, {0: LOAD, 1: k % 9, 2: STORE, 3: 24 + k % 700, 4: LOAD, 5: 0, 6: ADD, 7: 3, 8: ADD, 9: 20,
                        10: STORE, 11: 3, 12: JMP, 13: 0, 20: 1 + 2 * (k % 3)}) for k in range(num_vms)]
    return W.from_programs(W.ISA_CLASSIC, progs, n, [[]] * num_vms, ell=0, s=1)


# budgets on both sides of the fewest transitions traces are compiled for
# (8,192 after the first pass)
CASES = {
    "classic-n7": (lambda: _uniform(1, 6000, 1, 7), dict(first_pass=4), 8195),
    "classic-n1": (lambda: _uniform(2, 3000, 1, 1), dict(first_pass=4), 8196),
    "classic-n2": (lambda: _uniform(3, 3000, 1, 2), dict(first_pass=4), 8197),
    "classic-n64": (lambda: _uniform(4, 40000, 1, 64), dict(first_pass=4), 8196),
    "word-n31": (lambda: _uniform(5, 40000, 0, 31), dict(first_pass=1), 9000),
    "word-n64-lds64": (lambda: _uniform(6, 20000, 0, 64), dict(first_pass=16, lds_words=64), 8208),
    "classic-n33-w8": (lambda: _uniform(7, 40000, 1, 33, w=8), dict(first_pass=600), 9000),
    "word-n40-w29": (lambda: _uniform(8, 20000, 0, 40, w=29), dict(), 8300),
    "boundaries": (lambda: W.from_programs(1, _boundary_programs(41) * 20, 41, [[3, -4]] * 100, ell=2, s=2),
                   dict(first_pass=1), 9000),
    "uneven": (lambda: W.config3(num_vms=6000, seed=9), dict(lds_words=40, first_pass=576), 20000),
    # more survivors than one round of k_whole's lanes
    "uneven-many": (lambda: W.config3(num_vms=90000, seed=33), dict(first_pass=64), 8400),
    # sorted first (n of at most 512), and not
    "fig1": (lambda: W.fig1(num_vms=2000), dict(first_pass=64, lds_words=152), 30000),
    "wanderers-n512": (lambda: _wanderers(2000, 512), dict(first_pass=64), 8300),
    "wanderers-n513": (lambda: _wanderers(2000, 513), dict(first_pass=64), 8300),
    "wanderers": (lambda: _wanderers(700, 1024), dict(first_pass=64), 9000),
    # survivors that go to k_whole without traces: n of one to four lanes a wave,
    # and one word more than it takes; more survivors than its lanes
    "whole-n2048": (lambda: _wanderers(300, 2048), dict(first_pass=64), 4000),
    "whole-n2049": (lambda: _wanderers(300, 2049), dict(first_pass=64), 4000),
    "whole-n1": (lambda: _uniform(12, 1025, 1, 1), dict(first_pass=1), 700),
    "whole-n250-w16": (lambda: _uniform(13, 30000, 0, 250, w=16), dict(first_pass=8, lds_words=252), 4000),
    "whole-n1024-many": (lambda: _wanderers(9000, 1024), dict(first_pass=64), 1000),
    # transients in a pass of their own (memories in HBM, 1,024 transitions
    # left), with survivors for k_whole and for the work queue, and without
    "warm-whole": (lambda: W.config3(num_vms=9000, seed=30), dict(lds_words=0, first_pass=64), 1088),
    "warm-queue": (lambda: W.config3(num_vms=70000, seed=31), dict(first_pass=3), 2000),
    "no-warm": (lambda: W.config3(num_vms=9000, seed=32), dict(lds_words=0, first_pass=64), 1087),
    # whole in LDS from the start, c0's zero tails not stored yet: up to 8
    # machines a wave (8,192 on 256 CUs), and one more
    "direct-n3": (lambda: _uniform(15, 1000, 1, 3), dict(first_pass=4), 40),
    "direct-n63": (lambda: _uniform(16, 8192, 1, 63), dict(first_pass=4), 900),
    "first-n63": (lambda: _uniform(16, 8193, 1, 63), dict(first_pass=4), 900),
    "direct-word-n129-w8": (lambda: _uniform(17, 3000, 0, 127, w=8), dict(), 1500),
    "direct-n1023": (lambda: _wanderers(4097, 1023), dict(), 1000),
    # more of them than k_whole takes: the work queue steps them
    "wanderers-many": (lambda: _wanderers(40000, 1024), dict(first_pass=64), 8300),
}


@pytest.fixture(scope="module")
def R():
    import torch
    from paper_2604_12902_amd import rasp as R
    assert torch.cuda.is_available()
    return R


def _context(R, knobs, nbytes=1 << 30):
    c = R.Context(nbytes)
    c.set(R.RASP_OPT_SCHEDULE, 2)
    for k, v in knobs.items():
        c.set({"first_pass": R.RASP_OPT_FIRST_PASS, "lds_words": R.RASP_OPT_LDS_WORDS}[k], v)
    return c


@pytest.mark.parametrize("case", list(CASES) + ["states-classic", "states-word", "runs", "multi", "no-room", "graph", "noalloc"])
def test_traces_bit_exact(R, case):
    print("case:", case, flush=True)
    if case in CASES:
        make, knobs, budget = CASES[case]
        b = make()
        with _context(R, knobs) as c:
            h = c.load(b)
            c.run(h, budget)
            compare(c.fetch(h, mem=True), oracle.run(b, budget, threads=8, w=b.word_bits))
    elif case.startswith("states"):
        # i near INT32_MAX, odd, negative; a and memory at the int32 edges
        isa = 1 if case == "states-classic" else 0
        b = W.tiny_random(seed=50 + isa, num_vms=8000, isa=isa, max_m=6, max_n=30, max_ell=4, max_s=3, opcode_hi=10)
        st = _random_states(b, seed=51 + isa)
        with _context(R, dict(first_pass=2)) as c:
            h = c.load_state(b, dict(i=st.i, a=st.a, u0=st.u0, y0=st.y0, steps=st.steps, y=st.Y, mem=st.mem))
            c.run(h, 8200)
            oracle.advance(st, 8200)
            compare(c.fetch(h, mem=True), st)
    elif case == "runs":
        # one run's machines go on in the next
        b = W.config3(num_vms=3000, seed=10)
        with _context(R, dict(first_pass=100)) as c:
            h = c.load(b)
            for budget in (8500, 1, 8292, 4000):
                c.run(h, budget)
            compare(c.fetch(h, mem=True), oracle.run(b, 20793, threads=8))
    elif case == "multi":
        # several batches in one launch: the lists hold machines of all
        bs = [W.config3(num_vms=1000 + 77 * k, seed=20 + k) for k in range(3)]
        with _context(R, dict(first_pass=64)) as c:
            hs = [c.load(b) for b in bs]
            c.run_multi(hs, [9000, 2600, 9000])
            for h, b, budget in zip(hs, bs, (9000, 2600, 9000)):
                compare(c.fetch(h, mem=True), oracle.run(b, budget, threads=8))
    elif case in ("graph", "noalloc"):
        # the survivors' launches captured, and without an allocation
        b = _uniform(14, 20000, 1, 61)
        with _context(R, dict(first_pass=8)) as c:
            h = c.load(b)
            c.set(R.RASP_OPT_GRAPH, 1 if case == "graph" else 0)
            for k in range(3):
                (c.run if case == "graph" else lambda x, y: R.rasp_run_noalloc(c.handle, x, y))(h, 1500)
                c.sync(h)
            compare(c.fetch(h, mem=True), oracle.run(b, 4500, threads=8))
    else:
        # an arena with room for the load (32 bytes a machine of staging) but not
        # for the survivor list and the lists traces need (40 bytes): the run
        # goes without them
        progs = [[1, k % 5, 8, 0] if k % 3 else [1, 7, 4, 2] for k in range(1 << 20)]
        b = W.from_programs(W.ISA_CLASSIC, progs, 32, ell=0, s=1)
        room = R.rasp_batch_footprint(R.make_desc(b)) + 34 * b.N + (1 << 20)
        with _context(R, dict(first_pass=4), room) as c:
            h = c.load(b)
            c.run(h, 8200)
            compare(c.fetch(h), oracle.run(b, 8200, threads=8), mem=False)


# a load's waves walk 4 to 64 machines each, by the machines there are
@pytest.mark.parametrize("num_vms", [1, 5, 63, (8 << 16) - 1, 8 << 16, (16 << 16) + 3])
def test_load_groups_of_machines(R, num_vms):
    print("case: load", num_vms, flush=True)
    rng = np.random.Generator(np.random.PCG64(num_vms))
    m = rng.integers(0, 5, num_vms)
    words = rng.integers(-9, 9, int(2 * m.sum()), dtype=np.int32)
    off = W._offsets(2 * m)
    b = W.Batch(W.ISA_CLASSIC, words, off, rng.integers(8, 14, num_vms).astype(np.uint32), np.arange(num_vms, dtype=np.int32),
                np.arange(num_vms + 1, dtype=np.uint64), np.ones(num_vms, np.uint32), np.ones(num_vms, np.uint32))
    with R.Context(1 << 30) as c:
        h = c.load(b)
        compare(c.fetch(h, mem=True), oracle.run(b, 0))


# copies of host arrays below, at and above the sizes from which they go in
# chunks (512 KiB) and by way of the pinned area (256 KiB, 1 MiB in all)
@pytest.mark.parametrize("num_vms,n", [(64, 1024), (65537, 1), (131071, 1), (128, 1025), (3 << 18, 1), (10001, 1021)])
def test_state_round_trip_by_size(R, num_vms, n):
    print("case: round trip", num_vms, n, flush=True)
    rng = np.random.Generator(np.random.PCG64(num_vms + n))
    b = W.Batch(W.ISA_CLASSIC, np.zeros(0, np.int32), np.zeros(num_vms + 1, np.uint64), np.full(num_vms, n, np.uint32),
                np.zeros(0, np.int32), np.zeros(num_vms + 1, np.uint64), np.ones(num_vms, np.uint32),
                np.full(num_vms, 2, np.uint32))
    st = oracle.init(b)
    for k in ("i", "a"):
        setattr(st, k, rng.integers(-2 ** 31, 2 ** 31, num_vms).astype(np.int32))
    st.mem = rng.integers(-2 ** 31, 2 ** 31, st.mem.size).astype(np.int32)
    st.Y = rng.integers(-9, 9, st.Y.size).astype(np.int32)
    st.steps = rng.integers(0, 1000, num_vms).astype(np.uint64)
    with R.Context(1 << 30) as c:
        for _ in range(2):
            h = c.load_state(b, dict(i=st.i, a=st.a, u0=st.u0, y0=st.y0, steps=st.steps, y=st.Y, mem=st.mem))
            got = c.fetch(h, mem=True, digest=True)
            c.free(h)
            want = st.copy()
            oracle.advance(want, 0)
            compare(got, want)
            assert np.array_equal(got["mem_digest"], oracle.digest(want))
