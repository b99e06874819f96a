"""GPU parity where a launch's sizes or the arena come to their limits."""
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
