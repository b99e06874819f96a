"""GPU parity where a launch's sizes or the arena come to their limits."""
import numpy as np
import pytest

import oracle
from paper_2604_12902_amd import workloads as W
from test_gpu_parity import compare
from test_gpu_traces import _context

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    from paper_2604_12902_amd import rasp as R
    assert torch.cuda.is_available()
    return R


# a memory whose slots in LDS would take a multiple of 2^32 bytes a block: no
# survivor list of it goes to k_whole
@pytest.mark.parametrize("n", [(1 << 22) - 2, (1 << 22) - 1])
@pytest.mark.parametrize("graph", [0, 1])
def test_memories_far_beyond_a_slot(R, n, graph):
    print("case: memory", n, graph, flush=True)
    b = W.from_programs(W.ISA_CLASSIC, [[1, 5, 4, n - 1, 2, n - 1, 8, 2]], n, [[]], ell=0, s=1)
    with _context(R, dict(first_pass=8)) as c:
        c.set(R.RASP_OPT_GRAPH, graph)
        h = c.load(b)
        c.run(h, 200)
        compare(c.fetch(h, mem=True), oracle.run(b, 200))


# an arena with room for a batch but not for a dump of its memories: the fetch
# behind a run fails, and the batch loaded next is whole
@pytest.mark.parametrize("num_vms", [1500, 20000])
def test_load_after_a_fetch_without_room(R, num_vms):
    print("case: fetch without room", num_vms, flush=True)
    first = W.config3(num_vms=num_vms, seed=61)
    first.mem_words = np.full(num_vms, 1025, np.uint32)
    then = W.config3(num_vms=num_vms, seed=62)
    then.mem_words = np.full(num_vms, 1025, np.uint32)
    room = max(R.rasp_batch_footprint(R.make_desc(b)) for b in (first, then)) + 100 * num_vms + (1 << 20)
    room += 4 * max(first.prog.size + first.tape.size, then.prog.size + then.tape.size)
    with _context(R, dict(first_pass=64), room) as c:
        h = c.load(first)
        c.run(h, 30000)
        with pytest.raises(R.RaspError) as e:
            c.fetch(h, mem=True)
        assert e.value.code == R.RASP_E_NOMEM
        c.free(h)
        h = c.load(then)
        c.run(h, 3000)
        got = c.fetch(h, digest=True)
        want = oracle.run(then, 3000, threads=8)
        compare(got, want, mem=False)
        assert np.array_equal(got["mem_digest"], oracle.digest(want))


def _mixed(num_vms, wander, n):
    """Machines that run in nodes (a counted loop) and, every `wander`-th one
    (0: none), machines that store through a moving address."""
    LOAD, ADD, SUB, STORE, JPOS, JMP = 1, 2, 3, 4, 5, 8
    progs = []
    for k in range(num_vms):
        if wander and k % wander == 0:
            progs.append([LOAD, k % 9, STORE, 24 + k % 400, LOAD, 0, ADD, 7, ADD, 20, STORE, 7, JMP, 2,
                          0, 0, 0, 0, 0, 0, 2])
        else:
            progs.append([LOAD, 20000 + k % 50, SUB, 21, STORE, 22, LOAD, 1, STORE, 21, LOAD, 0, ADD, 22, SUB, 21,
                          STORE, 22, JPOS, 10, 0, 0, 0])
    return W.from_programs(W.ISA_CLASSIC, progs, n, [[]] * num_vms, ell=0, s=1)


# sorted survivors, with as many beside the nodes as send all of them to k_whole
# (one in 64), fewer, and none; and more of them than one round of it holds
@pytest.mark.parametrize("num_vms,wander", [(640, 64), (640, 100), (640, 0), (640, 1), (40000, 20)])
def test_sorted_survivors_together_or_apart(R, num_vms, wander):
    print("case: sorted", num_vms, wander, flush=True)
    b = _mixed(num_vms, wander, 480)
    with _context(R, dict(first_pass=64)) as c:
        h = c.load(b)
        c.run(h, 9000)
        compare(c.fetch(h, mem=True), oracle.run(b, 9000, threads=8))


# waves most of whose machines step in general from the start on, and waves
# with as many that do not; below and above the machines of a wave from which
# on they leave together; one list of both kinds of memory
@pytest.mark.parametrize("num_vms,wander,n", [(30000, 1, 480), (30000, 2, 480), (30000, 3, 480), (9000, 1, 480),
                                              (30000, 1, 900), (16000, 2, 900)])
def test_waves_of_machines_outside_nodes(R, num_vms, wander, n):
    print("case: crowd", num_vms, wander, n, flush=True)
    b = _mixed(num_vms, wander, n)
    with _context(R, dict(first_pass=64)) as c:
        h = c.load(b)
        c.run(h, 8600)
        compare(c.fetch(h, mem=True), oracle.run(b, 8600, threads=8))


# machines that read a tape longer than 64 words in a loop, then run in nodes
def test_waves_of_long_tapes(R):
    LOAD, ADD, STORE, JPOS, READ, JMP = 1, 2, 4, 5, 6, 8
    b = W.from_programs(W.ISA_CLASSIC, [[READ, 30, LOAD, 0, ADD, 30, JPOS, 0, LOAD, 1, ADD, 31, STORE, 31, JMP, 8]] * 30000,
                        100 + 4 * 7, [[1] * 200 + [-1] * 3] * 30000, ell=203, s=1)
    with _context(R, dict(first_pass=64)) as c:
        h = c.load(b)
        c.run(h, 8600)
        compare(c.fetch(h, mem=True), oracle.run(b, 8600, threads=8))


# memories in HBM, a budget below that of traces: survivor lists of up to two
# rounds of k_whole run their transients in a pass of their own, longer ones do
# not (16,384 on 256 CUs at n = 1,024: 57,000 machines of this population)
@pytest.mark.parametrize("num_vms", [40000, 57000, 90000])
def test_passes_before_short_and_long_lists(R, num_vms):
    print("case: passes", num_vms, flush=True)
    b = W.config3(num_vms=num_vms, seed=34)
    with _context(R, dict(first_pass=64)) as c:
        h = c.load(b)
        c.run(h, 1500)
        compare(c.fetch(h, mem=True), oracle.run(b, 1500, threads=8))


# more machines outside nodes than k_whole takes in a context with hot cells:
# the work queue steps them in HBM, whatever the slots
@pytest.mark.parametrize("num_vms,n,lds_words", [(40000, 900, 40), (70000, 480, 0), (70000, 480, 480)])
def test_work_queue_of_a_hot_cell_context(R, num_vms, n, lds_words):
    print("case: hot cells", num_vms, n, lds_words, flush=True)
    b = _mixed(num_vms, 1, n)
    with _context(R, dict(first_pass=576, lds_words=lds_words)) as c:
        c.set(R.RASP_OPT_HOT_CELLS, 32)
        c.set(R.RASP_OPT_PROFILE_STEPS, 512)
        h = c.load(b)
        c.run(h, 8900)
        compare(c.fetch(h, mem=True), oracle.run(b, 8900, threads=8))


# work lists with memories in HBM, of one machine to more waves than one block on
# every compute unit holds: each machine is some wave's
@pytest.mark.parametrize("num_vms", [1, 64, 65, 64 * 257, 64 * 4 * 256, 64 * 4 * 256 + 1, 64 * 4 * 300 + 7])
def test_work_lists_of_every_length(R, num_vms):
    print("case: work list", num_vms, flush=True)
    n = 2049 if num_vms < 20000 else 1030
    # (memories too large for k_whole, or more machines than it takes)
    b = _mixed(num_vms, 3, n)
    with _context(R, dict(first_pass=8)) as c:
        h = c.load(b)
        c.run(h, 150)
        compare(c.fetch(h, digest=True), oracle.run(b, 150, threads=8), mem=False)
