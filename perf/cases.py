"""The framework's work, as a list of cases with their inputs and exact results.

A case is one call that a program makes through
``paper_2208_11617_amd.binding``: a single launch of an operation over
Delta_n^m, several generations of an automaton, or one work-queue launch over
a mixed batch of jobs.  The single calls with the sizes 1024 (2-D and 3-D),
16384 (2-D) and 128 (4-D) are the benchmark's workloads; the job mix is its
serving stream's; the other sizes are odd ones between the smallest call and
those.

  listed()         the fixed cases
  draw(rng)        one more case of the same kinds and ranges
  prepare(case, seed)   inputs and outputs on the GPU, made from the seed
  run(state)       one pass through the public entry points
  work(case)       bytes and operations of one pass that cannot be avoided
  exact(case, seed)     the result in plain torch

Cells and elements outside the simplex are never written: outputs keep there
what they held before (zeros; drawn words for the hash, which reads no
input).  Input cells outside it hold whatever was drawn.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2208_11617_amd import binding as smap

# share of live cells at the start, per automaton (of 256)
DENSITY = {2: 77, 3: 51}
JOB_DENSITY = 64


def listed():
    return [
        # one Life step on a board that fits any cache: the launch is the cost
        {"name": "life_small", "kind": "step", "m": 2, "n": 200},
        # the 2-D accumulator, 0.5 M elements: short, still more than a launch
        {"name": "accum_2d", "kind": "accum", "m": 2, "n": 1024},
        # one Life step of the large board
        {"name": "life_large", "kind": "step", "m": 2, "n": 16384},
        # a run of Life, several generations a call: large board, full pass
        {"name": "life_run_large", "kind": "gens", "m": 2, "n": 16384, "steps": 32},
        # the same on an ordinary odd board with a part of a pass
        {"name": "life_run_mid", "kind": "gens", "m": 2, "n": 3001, "steps": 17},
        # one step of the 3-D automaton at the benchmark's size
        {"name": "ca3_large", "kind": "step", "m": 3, "n": 1024},
        # the same below the size from which the large tile is used, odd
        {"name": "ca3_mid", "kind": "step", "m": 3, "n": 383},
        # a run of the 3-D automaton at the benchmark's size: the heaviest call
        {"name": "ca3_run_large", "kind": "gens", "m": 3, "n": 1024, "steps": 16},
        # a short run on an ordinary odd box
        {"name": "ca3_run_mid", "kind": "gens", "m": 3, "n": 301, "steps": 8},
        # the 4-D hash of every element
        {"name": "hash_4d", "kind": "hash", "m": 4, "n": 128},
        # the distance matrix of 16385 points, upper triangle
        {"name": "edm_large", "kind": "edm", "m": 2, "n": 16384},
        # one launch of the serving loop: 96 mixed jobs of many sizes
        {"name": "queue_mix", "kind": "queue", "jobs": 96, "mix": 5},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    kind = rng.choice(["step", "step", "step", "gens", "gens", "gens", "accum", "hash", "edm", "queue"])
    if kind == "queue":
        return {"kind": "queue", "jobs": _log(rng, 2, 96), "mix": rng.randrange(1, 1 << 30)}
    if kind == "edm":
        return {"kind": "edm", "m": 2, "n": _log(rng, 64, 16384)}
    if kind in ("accum", "hash"):
        m = rng.choice([2, 3, 4])
        return {"kind": kind, "m": m, "n": _log(rng, *{2: (64, 8192), 3: (32, 600), 4: (8, 128)}[m])}
    m = rng.choice([2, 3])
    n = _log(rng, *{2: (64, 16384), 3: (32, 1024)}[m])
    if kind == "gens":
        return {"kind": "gens", "m": m, "n": n, "steps": rng.randint(2, 32 if m == 2 else 16)}
    return {"kind": "step", "m": m, "n": n}


def _jobs(case):
    """(m, n) of the batch's jobs: three of five 2-D with sides 64 to 4096, the others 3-D with 32 to 512."""
    rng = random.Random(case["mix"])
    return [(2, _log(rng, 64, 4096)) if rng.random() < 0.6 else (3, _log(rng, 32, 512)) for _ in range(case["jobs"])]


def _slots(jobs):
    """Byte offsets of the jobs' boxes in one arena (256-byte slots, as the serving loop places them)."""
    offs, at = [], 0
    for m, n in jobs:
        offs.append(at)
        at += ((n + 1) ** m + 255) // 256 * 256
    return offs, at


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _cells(count, density, seed):
    c = torch.randint(0, 256, (count,), dtype=torch.uint8, device="cuda", generator=_gen(seed))
    return c.lt_(density)


def _box(m, n):
    return (n + 1,) * m


def _words(m, n, seed):
    return torch.randint(0, 1 << 31, _box(m, n), dtype=torch.int32, device="cuda", generator=_gen(seed))


def _input(case, seed):
    kind, m, n = case["kind"], case.get("m"), case.get("n")
    if kind == "queue":
        return _cells(_slots(_jobs(case))[1], JOB_DENSITY, seed)
    if kind in ("step", "gens"):
        return _cells((n + 1) ** m, DENSITY[m], seed).view(_box(m, n))
    if kind == "accum":
        return _words(m, n, seed)
    if kind == "edm":
        return torch.rand((n + 1, 3), dtype=torch.float32, device="cuda", generator=_gen(seed))
    return None                                     # the hash reads nothing


def prepare(case, seed):
    kind, m, n = case["kind"], case.get("m"), case.get("n")
    src = _input(case, seed)
    if kind == "queue":
        jobs = _jobs(case)
        offs, total = _slots(jobs)
        out = torch.zeros(total, dtype=torch.uint8, device="cuda")
        calls = []
        for (jm, jn), o in zip(jobs, offs):
            size = (jn + 1) ** jm
            calls.append((jm, "ca2" if jm == 2 else "ca3", jn, src[o:o + size], out[o:o + size]))
        return {"kind": kind, "calls": calls, "in": src, "out": out}
    dtype = {"accum": torch.int32, "hash": torch.int32, "edm": torch.float32}.get(kind, torch.uint8)
    # the hash reads no input: its box starts with a program's earlier values, which the elements outside keep
    out = _words(m, n, seed) if kind == "hash" else torch.zeros(_box(m, n), dtype=dtype, device="cuda")
    op = {"accum": "accum", "hash": "hash", "edm": "edm"}.get(kind) or ("ca2" if m == 2 else "ca3")
    return {"kind": kind, "m": m, "n": n, "op": op, "steps": case.get("steps"), "in": src, "out": out}


def run(state):
    if state["kind"] == "queue":
        smap.queue_launch(state["calls"])
    elif state["kind"] == "gens":
        smap.map_launch_steps(state["m"], state["n"], state["op"], state["steps"], state["in"], state["out"])
    else:
        smap.map_launch(state["m"], state["n"], state["op"], state["in"], state["out"])
    return state["out"]


def work(case):
    kind = case["kind"]
    if kind == "queue":
        cells2 = sum(math.comb(n + m, m) for m, n in _jobs(case) if m == 2)
        cells3 = sum(math.comb(n + m, m) for m, n in _jobs(case) if m == 3)
        return {"bytes": 2 * (cells2 + cells3), "flops": 10 * cells2 + 28 * cells3}
    m, n = case["m"], case["n"]
    cells = math.comb(n + m, m)
    if kind == "accum":
        return {"bytes": 8 * cells, "flops": cells}
    if kind == "hash":
        return {"bytes": 4 * cells, "flops": (2 * m + 5) * cells}
    if kind == "edm":
        return {"bytes": 4 * cells + 12 * (n + 1), "flops": 9 * cells}
    per_cell = 10 if m == 2 else 28                 # neighbour sums and the rule
    return {"bytes": 2 * cells, "flops": per_cell * cells * case.get("steps", 1)}


def _inside(m, n, device="cuda"):
    r = torch.arange(n + 1, dtype=torch.int32, device=device)
    s = r
    for _ in range(m - 1):
        s = s.unsqueeze(-1) + r
    return s <= n


def _automaton(cells, m, n, steps):
    inside = _inside(m, n)
    x = cells.clone().mul_(inside)
    for _ in range(steps):
        s = x
        for d in range(m):                          # 3^m sums, one axis after another
            t = s.clone()
            t.narrow(d, 1, n).add_(s.narrow(d, 0, n))
            t.narrow(d, 0, n).add_(s.narrow(d, 1, n))
            s = t
        if m == 2:
            nxt = (s == 3) | ((s == 4) & (x == 1))
        else:
            nxt = (s == 6) | (((s == 7) | (s == 8)) & (x == 1))
        x = (nxt & inside).to(torch.uint8)
    return x


def _mul32(h, k):
    return (h * k) & 0xFFFFFFFF


def exact(case, seed):
    kind, m, n = case["kind"], case.get("m"), case.get("n")
    src = _input(case, seed)
    if kind == "queue":
        jobs = _jobs(case)
        offs, total = _slots(jobs)
        out = torch.zeros(total, dtype=torch.uint8, device="cuda")
        for (jm, jn), o in zip(jobs, offs):
            size = (jn + 1) ** jm
            out[o:o + size] = _automaton(src[o:o + size].view(_box(jm, jn)), jm, jn, 1).view(-1)
        return out
    if kind in ("step", "gens"):
        return _automaton(src, m, n, case.get("steps", 1))
    if kind == "accum":                             # below 2^31 before, uint32 after
        return (src + 1).mul_(_inside(m, n))
    if kind == "edm":                               # element (x1, x2): points x1 and n - x2
        p = src.double()
        out = torch.zeros((n + 1, n + 1), dtype=torch.float64, device="cuda")
        for c in range(3):
            out.add_((p[:, c].unsqueeze(0) - p[:, c].flip(0).unsqueeze(1)).square_())
        return out.sqrt_().mul_(_inside(2, n))
    r = torch.arange(n + 1, dtype=torch.int64, device="cuda")
    h = torch.full((1,) * m, 0x811C9DC5, dtype=torch.int64, device="cuda")
    for k in range(m):                              # FNV-1a over x_1 (the last axis) to x_m
        h = _mul32(h ^ r.view((-1,) + (1,) * k), 0x01000193)
    h = h ^ (h >> 16)
    h = _mul32(h, 0x85EBCA6B)
    h = h ^ (h >> 13)
    h = _mul32(h, 0xC2B2AE35)
    h = h ^ (h >> 16)
    return torch.where(_inside(m, n), h.to(torch.int32), _words(m, n, seed))
