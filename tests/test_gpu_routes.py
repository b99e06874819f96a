"""Which way a run is launched on both sides of each rule, by RASP_OPT_ROUTE, and
that it is bit-exact there."""
import pytest

import oracle
from paper_2604_12902_amd import workloads as W
from test_gpu_parity import compare
from test_gpu_traces import _context, _uniform, _wanderers

pytestmark = pytest.mark.gpu

FIRST, DIRECT, WHOLE, PASS, TRACES, SORTED, HOT, NO_ROOM = (1 << k for k in range(8))


@pytest.fixture(scope="module")
def R():
    import torch
    from paper_2604_12902_amd import rasp as R
    assert torch.cuda.is_available()
    assert (R.RASP_ROUTE_FIRST, R.RASP_ROUTE_DIRECT, R.RASP_ROUTE_WHOLE, R.RASP_ROUTE_PASS, R.RASP_ROUTE_TRACES,
            R.RASP_ROUTE_SORTED, R.RASP_ROUTE_HOT_CELLS, R.RASP_ROUTE_NO_ROOM) == (
                FIRST, DIRECT, WHOLE, PASS, TRACES, SORTED, HOT, NO_ROOM)
    return R


# (population, first pass, options, budget, route); None: eight machines a
# wave of four waves a CU, the most that run whole in LDS from the start
CASES = {
    "direct": (lambda most: _uniform(16, most, 1, 63), 4, {}, 900, DIRECT),
    "not-direct": (lambda most: _uniform(16, most + 1, 1, 63), 4, {}, 900, FIRST | WHOLE),
    "direct-hot": (lambda most: _uniform(16, 2000, 1, 63), 4, dict(HOT_CELLS=8), 900, FIRST | HOT),
    "whole": (lambda most: _wanderers(most + 1, 2048), 64, {}, 400, FIRST | WHOLE),
    "whole-pass": (lambda most: _wanderers(most + 1, 2048), 64, {}, 1088, FIRST | WHOLE | PASS),
    "not-whole": (lambda most: _wanderers(300, 2049), 64, {}, 4000, FIRST),
    "traces": (lambda most: _wanderers(500, 1024), 64, {}, 8256, FIRST | WHOLE | TRACES | PASS),
    "traces-late": (lambda most: _wanderers(500, 1024), 512, {}, 8704, FIRST | WHOLE | TRACES),
    "too-short": (lambda most: _wanderers(500, 1024), 64, {}, 8255, DIRECT),
    "too-large": (lambda most: _wanderers(500, 1025), 64, {}, 8256, DIRECT),
    "sorted": (lambda most: _wanderers(500, 512), 64, {}, 8256, FIRST | WHOLE | TRACES | SORTED),
    "not-sorted": (lambda most: _wanderers(500, 513), 64, {}, 8256, FIRST | WHOLE | TRACES | PASS),
    "off": (lambda most: _wanderers(most + 1, 512), 64, dict(TRACES=0), 8256, FIRST | WHOLE | PASS),
    "off-direct": (lambda most: _wanderers(500, 512), 64, dict(TRACES=0), 8256, DIRECT),
    "hot": (lambda most: _wanderers(500, 1024), 576, dict(HOT_CELLS=32), 9000, FIRST | WHOLE | TRACES),
    "hot-off": (lambda most: _wanderers(500, 1024), 576, dict(HOT_CELLS=32, TRACES=0), 9000, FIRST | HOT),
    "plain": (lambda most: _wanderers(500, 1024), 64, dict(SCHEDULE=1), 8256, 0),
    "no-first-pass": (lambda most: _uniform(16, 2000, 1, 63), 0, {}, 9000, 0),
    "graph": (lambda most: _wanderers(500, 1024), 64, dict(GRAPH=1), 8256, FIRST | WHOLE),
}


@pytest.mark.parametrize("case", list(CASES) + ["noalloc", "no-room"])
def test_route(R, case):
    print("case:", case, flush=True)
    if case == "noalloc":
        b, budget, want, room, opts, first = _wanderers(500, 1024), 8256, FIRST | WHOLE, 1 << 30, {}, 64
    elif case == "no-room":
        # room for the load and the survivor list (4 bytes a machine), not for
        # the lists of traces (52)
        progs = [[1, k % 5, 8, 0] if k % 3 else [1, 7, 4, 2] for k in range(1 << 20)]
        b, budget, want, opts, first = W.from_programs(W.ISA_CLASSIC, progs, 32, ell=0, s=1), 8200, FIRST | WHOLE | NO_ROOM, {}, 4
        room = R.rasp_batch_footprint(R.make_desc(b)) + 34 * b.N + (1 << 20)
    else:
        make, first, opts, budget, want = CASES[case]
        room = 1 << 30
    with _context(R, dict(first_pass=first), room) as c:
        cus = R.rasp_device_info(c.handle)["compute_units"]
        if case in CASES:
            b = make(8 * 4 * cus)
        for k, v in opts.items():
            c.set(getattr(R, "RASP_OPT_" + k), v)
        h = c.load(b)
        if case == "noalloc":
            R.rasp_run_noalloc(c.handle, h, budget)
        else:
            c.run(h, budget)
        assert c.get(R.RASP_OPT_ROUTE) == want
        mem = case != "no-room"
        compare(c.fetch(h, mem=mem), oracle.run(b, budget, threads=8, w=b.word_bits), mem=mem)


def test_options(R):
    with R.Context(64 << 20) as c:
        assert c.get(R.RASP_OPT_TRACES) == 1
        for option, value in ((R.RASP_OPT_TRACES, 2), (R.RASP_OPT_TRACES, -1), (R.RASP_OPT_ROUTE, 0)):
            with pytest.raises(R.RaspError) as e:
                c.set(option, value)
            assert e.value.code == R.RASP_E_INVAL


# traces on a share of the compute units
@pytest.mark.parametrize("cus", [(0, 64), (192, 64), (0, 128)])
@pytest.mark.parametrize("n", [480, 900])
def test_traces_on_a_share(R, cus, n):
    print("case: share", cus, n, flush=True)
    b = _wanderers(600, n)
    u = _uniform(5, 1500, 1, 64)
    with R.Context(1 << 30, cus=cus) as c:
        for batch in (b, u):
            h = c.load(batch)
            c.run(h, 8600)
            assert c.get(R.RASP_OPT_ROUTE) & TRACES
            compare(c.fetch(h, mem=True), oracle.run(batch, 8600, threads=8))


# a trial over the first machines of a large batch takes the way of the whole
# batch; hot cells are tried without traces; a batch too short for traces, and
# a context without them, is searched as it is
@pytest.mark.parametrize("num_vms,part,budget,opts,want,never", [
    (40000, 3000, 1500, {}, FIRST | WHOLE | PASS, DIRECT | TRACES),
    (2000, 1000, 1500, {}, DIRECT, TRACES | HOT),
    (20000, 2000, 9000, {}, FIRST | TRACES | HOT, DIRECT | NO_ROOM),
    (20000, 2000, 9000, dict(TRACES=0), FIRST | HOT, DIRECT | TRACES | NO_ROOM),
])
def test_autotune_takes_the_way_of_the_whole_batch(R, num_vms, part, budget, opts, want, never):
    print("case: autotune", num_vms, part, budget, opts, flush=True)
    b = W.config3(num_vms=num_vms, seed=71)
    with R.Context(1 << 30) as c:
        for k, v in opts.items():
            c.set(getattr(R, "RASP_OPT_" + k), v)
        h = c.load(b)
        chosen = R.rasp_autotune(c.handle, h, budget, max_vms=part)
        print("chose", chosen, flush=True)
        route = c.get(R.RASP_OPT_ROUTE)
        assert route & want == want and route & never == 0, route
        assert chosen["traces"] == c.get(R.RASP_OPT_TRACES)
        c.run(h, budget)
        assert (c.get(R.RASP_OPT_ROUTE) & HOT != 0) == (chosen["hot_cells"] != 0)
        compare(c.fetch(h, mem=True), oracle.run(b, budget, threads=8))
