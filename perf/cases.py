"""Performance cases of librasp: what programs do with it, through the public
binding (``rasp.Context``, ``rasp_*``, ``serving.Server``).

One pass takes a batch of machines through the whole path: load (c0 from the
packed programs and inputs), run to the budget, fetch every per-machine result,
free.  Inputs are synthetic populations of the sizes this repository's
workloads, tests and benchmark use:

  uniform  random programs of m instructions (plain-small, plain-scale)
  uneven   programs of 8..512 instructions in memories of 64..1,024 words
  fig1     Sec. 3 word-RASP programs of 100 terminals, n = 250
  beaver   App. B's search population: 120 terminals, w = 29, arrays zero
  rollouts counted-loop array programs, n = 2,048, tapes of 1,024 words

Ways of driving the library ("mode"):

  device   descriptor and results in device memory (the benchmark's step)
  host     numpy arrays in, numpy arrays out (the README's example)
  inflight several batches at once, each on its own CU share and host thread
  serve    requests through serving.Server (host arrays, epochs, async fetches)
  resume   run, checkpoint to the host, load the state again, run on

"tuned" cases carry the scheduling knobs rasp_autotune chooses for their
population, which a program keeps and sets on its context; the others run with
the library's defaults.
"""
from __future__ import annotations

import math
import threading

import numpy as np
import torch

from paper_2604_12902_amd import rasp as R
from paper_2604_12902_amd import search, serving
from paper_2604_12902_amd import workloads as W

KNOBS = {"lds_words": R.RASP_OPT_LDS_WORDS, "first_pass": R.RASP_OPT_FIRST_PASS, "epoch": R.RASP_OPT_EPOCH,
         "waves_per_cu": R.RASP_OPT_WAVES_PER_CU, "hot_cells": R.RASP_OPT_HOT_CELLS,
         "profile_steps": R.RASP_OPT_PROFILE_STEPS, "misfit_waves": R.RASP_OPT_MISFIT_WAVES}
# the knobs rasp_autotune settles on for each population
TUNED = {"uneven": dict(lds_words=40, first_pass=576, epoch=256, hot_cells=32, profile_steps=512, misfit_waves=6),
         "fig1": dict(lds_words=152, first_pass=64, epoch=256),
         "rollouts": dict(lds_words=0, first_pass=64, epoch=256)}
FIELDS = ("status", "steps", "i", "a", "u0", "y0", "y")
POOL = 2048                              # distinct programs the fig1 and beaver populations are drawn from
ROLLOUT_POOL = 128


def listed():
    return [
        # the smallest call in use: a smoke test's thousand tiny machines, where launches and waits count
        dict(name="small 1K device", mode="device", family="uniform", N=1024, m=16, n=32, ell=8, s=256,
             budget=256, digest=True),
        # plain-small as the README drives it: host arrays in and out
        dict(name="small 4K host", mode="host", family="uniform", N=4096, m=16, n=32, ell=8, s=256,
             budget=256, digest=True),
        # an odd mid-sized request: memories that are no power of two, 16-bit words
        dict(name="ragged 100K w16", mode="device", family="uniform", N=100003, m=50, n=251, ell=17, s=5,
             budget=4096, digest=True, word_bits=16),
        # plain-scale: a million short programs, a few of which run to the budget
        dict(name="plain-scale 1M", mode="device", family="uniform", N=1 << 20, m=64, n=256, ell=32, s=16,
             budget=4096, digest=False),
        # a served request's shape with an untuned context: memories stay in HBM
        dict(name="uneven 50K untuned", mode="device", family="uneven", N=50021, budget=16384, digest=True),
        # the benchmark's population, one batch at a time on the whole chip
        dict(name="uneven 4M tuned", mode="device", family="uneven", N=1 << 22, budget=65536, digest=False,
             tuned=True),
        # the benchmark's headline way of running it: four batches on quarters of the chip
        dict(name="uneven 4x1M in flight", mode="inflight", family="uneven", N=1 << 20, budget=65536,
             digest=True, tuned=True, inflight=4),
        # the paper's Sec. 3 evaluation, whose loops run to the budget
        dict(name="fig1 256K tuned", mode="device", family="fig1", N=1 << 18, budget=400000, digest=True,
             tuned=True),
        # one round of the busy-beaver search (narrow words, few long runners)
        dict(name="beaver 64K w29", mode="device", family="beaver", N=1 << 16, budget=200000, digest=True,
             word_bits=29),
        # array programs with large memories and tapes
        dict(name="rollouts 64K tuned", mode="device", family="rollouts", N=1 << 16, budget=1 << 20,
             digest=True, tuned=True),
        # the serving loop: a burst of requests of mixed size and family
        dict(name="serve 12 requests", mode="serve", family="mixed", N=1024, N_hi=32768, requests=12,
             budget=16384, epoch=4096, digest=True),
        # checkpoint and resume: whole configurations to the host and back
        dict(name="resume 20K", mode="resume", family="uneven", N=20011, budget=2048, digest=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the listed families, sizes over their whole ranges."""
    kind = rng.choice(("uniform", "uniform", "uneven", "uneven", "fig1", "beaver", "rollouts", "host", "serve",
                       "resume", "inflight"))
    if kind in ("uniform", "host"):
        m = _log(rng, 8, 64)
        n = rng.choice((2 * m + rng.randrange(0, 64), 1 << (2 * m - 1).bit_length()))
        return dict(mode="device" if kind == "uniform" else "host", family="uniform",
                    N=_log(rng, 1000, 1 << 20 if kind == "uniform" else 1 << 15), m=m, n=n,
                    ell=rng.randrange(0, 33), s=_log(rng, 1, 256) if m <= 16 else _log(rng, 1, 16),
                    budget=_log(rng, 64, 4096), digest=rng.random() < 0.5,
                    word_bits=rng.choice((32, 32, 16, 29)))
    if kind == "uneven":
        tuned = rng.random() < 0.6
        return dict(mode="device", family="uneven", N=_log(rng, 2000, 1 << 21 if tuned else 1 << 17),
                    budget=_log(rng, 4096, 65536), digest=rng.random() < 0.5, tuned=tuned)
    if kind == "fig1":
        return dict(mode="device", family="fig1", N=_log(rng, 4096, 1 << 18), budget=_log(rng, 20000, 400000),
                    digest=True, tuned=True)
    if kind == "beaver":
        return dict(mode="device", family="beaver", N=_log(rng, 4096, 1 << 16), budget=_log(rng, 20000, 200000),
                    digest=True, word_bits=rng.choice((29, 24)))
    if kind == "rollouts":
        return dict(mode="device", family="rollouts", N=_log(rng, 2048, 1 << 16), budget=1 << 20, digest=True,
                    tuned=True)
    if kind == "serve":
        return dict(mode="serve", family="mixed", N=1024, N_hi=_log(rng, 2048, 32768),
                    requests=rng.randrange(3, 13), budget=_log(rng, 4096, 16384), epoch=4096, digest=True)
    if kind == "resume":
        return dict(mode="resume", family="uneven", N=_log(rng, 2000, 20000), budget=_log(rng, 512, 2048),
                    digest=True)
    return dict(mode="inflight", family="uneven", N=_log(rng, 1 << 16, 1 << 20), budget=_log(rng, 16384, 65536),
                digest=True, tuned=True, inflight=rng.choice((2, 4)))


# ---- populations -----------------------------------------------------------------------

_pools = {}


def _pool(family):
    """Distinct lowered programs (and arities) a population is drawn from."""
    if family not in _pools:
        if family == "fig1":
            b = W.fig1(num_vms=POOL)
        elif family == "beaver":
            b, _, _ = search.round_batch(0, 0, POOL, 120, 29, 1)
        else:
            b = W.config4(num_vms=ROLLOUT_POOL, num_distinct=ROLLOUT_POOL)
        _pools[family] = ([b.prog[b.prog_off[v]:b.prog_off[v + 1]] for v in range(b.N)],
                          np.diff(b.tape_off.astype(np.int64)))
    return _pools[family]


def _host_batch(case, seed):
    """A workloads.Batch of the case (families generated on the host)."""
    f, N = case["family"], case["N"]
    rng = np.random.Generator(np.random.PCG64(seed))
    if f == "uniform":
        n, wb = case["n"], case.get("word_bits", 32)
        hi = min(n, 1 << (wb - 1))
        b = W._uniform_batch(N, case["m"], 9, hi, n, case["ell"], -100, 100, case["s"], seed, case["budget"],
                             "uniform")
        b.word_bits = wb
        return b
    if f == "uneven":
        return W.config3(seed=seed, num_vms=N, budget=case["budget"])
    progs, arity = _pool(f)
    pick = rng.integers(0, len(progs), N)
    prog = np.concatenate([progs[k] for k in pick])
    off = W._offsets([len(progs[k]) for k in pick])
    if f == "rollouts":
        ell, n, s = W.ROLLOUT_ARRAY, W.ROLLOUT_MEM, W.ROLLOUT_OUT
        tape = rng.integers(-(1 << 15), 1 << 15, size=(N, ell), dtype=np.int32).reshape(-1)
        toff, isa = np.arange(N + 1, dtype=np.uint64) * np.uint64(ell), W.ISA_CLASSIC
    else:
        ell, n, s, isa = W.FIG1_ELL, W.FIG1_N, W.FIG1_S, W.ISA_WORD
        toff = W._offsets(arity[pick])
        tape = rng.integers(-(1 << 31), 1 << 31, size=int(toff[-1])).astype(np.int32)
    full = np.full(N, 1, np.uint32)
    return W.Batch(isa, prog, off, full * np.uint32(n), tape, toff, full * np.uint32(ell), full * np.uint32(s),
                   budget=case["budget"], name=f, word_bits=case.get("word_bits", 32))


def _device_arrays(case, seed):
    """(isa, arrays of the descriptor in device memory)."""
    f, N, dev = case["family"], case["N"], "cuda"
    if f not in ("uniform", "uneven"):
        b = _host_batch(case, seed)
        d = R.make_desc(b, torch.device(dev))
        names = ("prog", "prog_off", "mem_words", "tape", "tape_off", "tape_cap", "out_cap")
        return b.isa, dict(zip(names, d.keep))
    g = torch.Generator(dev).manual_seed(seed)
    rnd = dict(generator=g, device=dev)
    i32 = torch.int32
    if f == "uniform":
        m, n, ell, s = case["m"], case["n"], case["ell"], case["s"]
        hi = min(n, 1 << (case.get("word_bits", 32) - 1))
        prog = torch.stack([torch.randint(0, 9, (N, m), dtype=i32, **rnd),
                            torch.randint(0, hi, (N, m), dtype=i32, **rnd)], dim=2).reshape(-1)
        poff = torch.arange(N + 1, device=dev) * (2 * m)
        words = torch.full((N,), n, dtype=i32, device=dev)
    else:                                # the law of workloads.config3
        ell, s = 32, 16
        L = torch.exp(torch.rand(N, dtype=torch.float64, **rnd) * math.log(513 / 8) + math.log(8)).long().clamp(max=512)
        words = torch.exp(torch.rand(N, dtype=torch.float64, **rnd) * math.log(1025 / 64) + math.log(64)).long()
        words = torch.maximum(words.clamp(max=1024), 2 * L)
        halt = (torch.rand(N, **rnd) * L).long()
        poff = torch.zeros(N + 1, dtype=torch.int64, device=dev)
        torch.cumsum(2 * L, 0, out=poff[1:])
        prog = torch.empty(int(poff[-1]), dtype=i32, device=dev)
        for c in range(0, N, 1 << 18):
            Lc = L[c:c + (1 << 18)]
            first = poff[c:c + Lc.numel()] // 2
            tot, base = int(Lc.sum()), int(first[0])
            vm = torch.repeat_interleave(torch.arange(Lc.numel(), device=dev), Lc)
            k = torch.arange(tot, device=dev) - (first - base)[vm]
            Lv = Lc[vm]
            ops = torch.randint(1, 9, (tot,), dtype=i32, **rnd)
            ops[k == halt[c:c + Lc.numel()][vm]] = W.HALT
            u = torch.rand(tot, dtype=torch.float64, **rnd)
            tgt = torch.where(torch.rand(tot, **rnd) < 0.15, (u * (k + 1)).long(), k + 1 + (u * (Lv - k)).long())
            data = (torch.rand(tot, dtype=torch.float64, **rnd) * words[c:c + Lc.numel()][vm]).long()
            opd = torch.where((ops == W.JMP) | (ops == W.JPOS), 2 * tgt, data)
            opd[ops == W.HALT] = 0
            prog[2 * base:2 * (base + tot)] = torch.stack([ops, opd.to(i32)], dim=1).reshape(-1)
        words = words.to(i32)
    tape = torch.randint(-100, 101, (max(1, N * ell),), dtype=i32, **rnd)
    return W.ISA_CLASSIC, dict(prog=prog, prog_off=poff, mem_words=words, tape=tape,
                               tape_off=torch.arange(N + 1, device=dev) * ell,
                               tape_cap=torch.full((N,), ell, dtype=i32, device=dev),
                               out_cap=torch.full((N,), s, dtype=i32, device=dev))


# ---- states and passes -----------------------------------------------------------------

def _arena(case, words):
    """Arena bytes for a batch of N machines with `words` words in all."""
    hot = 96 if case.get("tuned") else 16
    return int((4 * words + (96 + hot) * case["N"]) * 1.06) + (64 << 20)


def _set_knobs(ctx, case):
    if case.get("tuned"):
        for k, v in TUNED[case["family"]].items():
            ctx.set(KNOBS[k], v)


def _outs(N, ny, digest):
    t = dict(status=torch.uint8, steps=torch.int64, i=torch.int32, a=torch.int32, u0=torch.int32, y0=torch.int32)
    out = {k: torch.zeros(N, dtype=d, device="cuda") for k, d in t.items()}
    out["y"] = torch.zeros(max(1, ny), dtype=torch.int32, device="cuda")
    if digest:
        out["mem_digest"] = torch.zeros(N, dtype=torch.int64, device="cuda")
    return out


_shares = {}                             # contexts on CU shares, kept by the program between batches


def _share_contexts(case, arena):
    n = case["inflight"]
    key = (n, case["N"])
    if key not in _shares:
        for old in _shares.pop(next(iter(_shares), None), []):
            old.close()
        cus = torch.cuda.get_device_properties(0).multi_processor_count
        # room beside the space of an earlier, slightly smaller batch
        _shares[key] = [R.Context(int(arena * 2.2), cus=R.cu_share(k, n, cus)) for k in range(n)]
        for c in _shares[key]:
            _set_knobs(c, case)
    return _shares[key]


def prepare(case, seed):
    mode, N = case["mode"], case["N"]
    st = dict(case=case)
    if mode in ("device", "inflight"):
        parts = []
        for k in range(case.get("inflight", 1)):
            isa, arrs = _device_arrays(case, seed * 16 + k)
            desc = R.desc_from_arrays(isa, N, flags=R.RASP_DESC_DEVICE_PTRS,
                                      word_bits=case.get("word_bits", 32), **arrs)
            ny = int(arrs["out_cap"].sum())
            words = int(((arrs["mem_words"].long() + 3) // 4 * 4 + arrs["tape_cap"]).sum()) + ny
            parts.append((desc, _outs(N, ny, case["digest"]), words))
        arena = _arena(case, max(p[2] for p in parts))
        torch.cuda.synchronize()
        if mode == "device":
            st["ctx"] = R.Context(arena)
            _set_knobs(st["ctx"], case)
            st["desc"], st["out"] = parts[0][:2]
        else:
            st["ctxs"] = _share_contexts(case, arena)
            st["parts"] = parts
    elif mode == "serve":
        # the same request shapes for every seed, machines of their own
        reqs = serving.poisson_requests(case["requests"], 1.0, size_lo=case["N"], size_hi=case["N_hi"],
                                        budget_lo=case["epoch"], budget_hi=case["budget"], generate=False)
        for q in reqs:
            q.arrival = 0.0
            q.batch = serving.make_batch(q.config, q.size, q.budget, seed * 1009 + q.rid)
        st["reqs"] = reqs
        cap = sum(4 * q.batch.footprint_words() + 128 * q.size + 4096 for q in reqs)
        st["ctx"] = R.Context(2 * cap + (768 << 20))
        st["server"] = serving.Server(serving.RaspExecutor(st["ctx"]), cap, epoch=case["epoch"])
    else:
        st["batch"] = _host_batch(case, seed)
        words = st["batch"].footprint_words() + 3 * N
        st["ctx"] = R.Context((3 if mode == "resume" else 2) * _arena(case, words) + (192 << 20))
    return st


def _device_pass(ctx, desc, out, budget):
    h = R.rasp_load_batch(ctx.handle, desc)
    R.rasp_run(ctx.handle, h, budget)
    R.rasp_fetch_outputs_into(ctx.handle, h, out, device=True)
    R.rasp_free_batch(ctx.handle, h)


def run(st):
    case = st["case"]
    mode, budget = case["mode"], case["budget"]
    if mode == "device":
        _device_pass(st["ctx"], st["desc"], st["out"], budget)
        return st["out"]
    if mode == "inflight":
        errors = []

        def drive(ctx, desc, out):
            try:
                _device_pass(ctx, desc, out, budget)
            except Exception as e:       # raised again below
                errors.append(e)
        threads = [threading.Thread(target=drive, args=(c, p[0], p[1])) for c, p in zip(st["ctxs"], st["parts"])]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        if errors:
            raise errors[0]
        return [p[1] for p in st["parts"]]
    if mode == "serve":
        st["server"].serve(st["reqs"])
        return {k: np.concatenate([q.result[k] for q in st["reqs"]]) for k in FIELDS + ("mem_digest",)}
    ctx = st["ctx"]
    h = ctx.load(st["batch"])
    if mode == "host":
        ctx.run(h, budget)
        out = ctx.fetch(h, digest=case["digest"])
        ctx.free(h)
        return out
    ctx.run(h, budget // 2)
    saved = ctx.fetch(h, mem=True)
    ctx.free(h)
    h = ctx.load_state(st["batch"], saved)
    ctx.run(h, budget - budget // 2)
    out = ctx.fetch(h, digest=case["digest"])
    ctx.free(h)
    return out


# ---- what a pass cannot do without -------------------------------------------------------

def work(case):
    """Input words, the words of c0 and the results each moved once; one
    operation a transition (the populations' mean transitions per machine)."""
    N, b, f = case["N"], case["budget"], case["family"]
    if f == "mixed":
        lo, hi = case["N"], case["N_hi"]
        N = int(case["requests"] * (hi - lo) / math.log(hi / lo)) if hi > lo else case["requests"] * lo
        words, steps = 700, 0.035 * b
    elif f == "uniform":
        words, steps = 2 * case["m"] + case["ell"] + case["s"], min(b, 4.5 + 0.0057 * b)
    elif f == "uneven":
        words, steps = 243 + 32 + 16, 0.11 * b
    elif f == "fig1":
        words, steps = 160 + 10 + 2, 0.24 * b
    elif f == "beaver":
        words, steps = 170 + 10 + 2, 0.047 * b
    else:
        words, steps = 500 + 2 * 1024, 140000
    N *= case.get("inflight", 1)
    host = 2 * 420 if case["mode"] == "resume" else 0
    return {"bytes": float(N * (4 * (2 * words + host) + 25)), "flops": float(max(1.0, N * steps))}


def exact(case, seed):
    """The results by a plain numpy interpreter of the machine's case table
    (classic instruction set), for the small populations; whole numbers."""
    if case["mode"] not in ("host", "device") or case["family"] != "uniform" or case["N"] * case["budget"] > 1 << 21:
        return None
    if case["mode"] == "host":
        b = _host_batch(case, seed)
        prog, tape = b.prog, b.tape
    else:
        _, arrs = _device_arrays(case, seed * 16)
        prog, tape = arrs["prog"].cpu().numpy(), arrs["tape"].cpu().numpy()
    N, n, m, ell, s = case["N"], case["n"], case["m"], case["ell"], case["s"]
    half = 1 << (case.get("word_bits", 32) - 1)
    M = np.zeros((N, n), np.int64)
    M[:, :2 * m] = prog.reshape(N, 2 * m)
    T = np.zeros((N, ell + 1), np.int64)
    T[:, :ell] = tape[:N * ell].reshape(N, ell)
    Y = np.zeros((N, s + 1), np.int64)
    i, a, u0, y0, steps = (np.zeros(N, np.int64) for _ in range(5))
    halted = np.zeros(N, bool)
    v = np.arange(N)
    wrap = lambda x: (x + half) % (2 * half) - half  # noqa: E731
    for k in range(case["budget"] + 1):
        o, j = M[v, i[v] % n], M[v, wrap(i[v] + 1) % n]
        taken = (o == 8) | ((o == 5) & (a[v] > 0))
        fixed = (o < 1) | (o > 8) | ((o == 6) & (u0[v] >= ell)) | (taken & (j == i[v]))
        halted[v[fixed]] = True
        v, o, j, taken = v[~fixed], o[~fixed], j[~fixed], taken[~fixed]
        if k == case["budget"] or v.size == 0:
            break
        d = M[v, j % n]
        st, rd, pr = o == 4, o == 6, (o == 7) & (y0[v] < s)
        M[v[st], j[st] % n] = a[v[st]]
        M[v[rd], j[rd] % n] = T[v[rd], u0[v[rd]]]
        Y[v[pr], y0[v[pr]]] = d[pr]
        u0[v] += rd
        y0[v] += pr
        a[v] = np.where(o == 1, j, wrap(a[v] + np.where(o == 2, d, 0) - np.where(o == 3, d, 0)))
        i[v] = np.where(taken, j, wrap(i[v] + 2))
        steps[v] += 1
    out = dict(status=halted.astype(np.uint8), steps=steps, i=i, a=a, u0=u0, y0=y0, y=Y[:, :s].reshape(-1))
    if case["digest"]:
        h = np.full(N, 0xcbf29ce484222325, np.uint64)
        for c in M.astype(np.int32).view(np.uint8).reshape(N, -1).T if n else ():
            h = (h ^ c) * np.uint64(0x100000001b3)
        out["mem_digest"] = h if case["mode"] == "host" else h.view(np.int64)
    if case["mode"] == "host":           # the binding's types
        for name, t in (("steps", np.uint64), ("u0", np.uint32), ("y0", np.uint32)):
            out[name] = out[name].astype(t)
    for name in ("i", "a", "y"):
        out[name] = out[name].astype(np.int32)
    if case["mode"] == "device":
        for name in ("u0", "y0"):
            out[name] = out[name].astype(np.int32)
    return out
