"""What a user has this framework do, as timed cases: checked jobs through the
public entry points (`paper_2401_04701_amd.hr`), from a one-block reduction to
label propagation over 2^25 edges.

A case is a dict of plain values.  `prepare` makes what the user's program
holds before the call (its data on the device, the checking context with the
buffers' shadow memory, a batch's job table); `run` is one checked job:
clear the checker's state, the job's checked launches with their launch
boundaries, and the report.  The outputs are the flagged set (a mask over the
words of every monitored buffer and of every block's LDS), the warning bits,
and the program's own results wherever they have one defined value: cells and
labels that a race reaches have none, and only the flagged set is returned.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import synth_inputs as si
from paper_2401_04701_amd import examples, hr

RMAT = (0.57, 0.19, 0.19)            # quadrant shares of the R-MAT graphs
GRID_LAUNCHES, GRAPH_LAUNCHES = 20, 10
MAPS = {"rowmajor": None, "4x4": (2, 2), "8x2": (3, 1)}


def listed():
    return [
        # one block's LDS tree reduction: the smallest call, where the cost is
        # the chain of launches, copies and round trips around one kernel
        {"name": "reduce_one_block", "kind": "reduce", "n": 512, "threads": 256, "blocks": 1,
         "drop": -1},
        # a grid of the largest reductions, with one step's barrier missing:
        # LDS checking over many blocks, and a report full of LDS races
        {"name": "reduce_grid_dropped", "kind": "reduce", "n": 2048, "threads": 1024,
         "blocks": 512, "drop": 5},
        # a small job run alone from nothing (its own context, shadow memory,
        # launches, report, release): the path of a script that checks one kernel
        {"name": "job_alone_stencil", "kind": "job", "pattern": "jacobi", "blocks": 100,
         "threads": 256, "seeded": False, "static": False},
        # a ragged grid, race-free: an ordinary program under test
        {"name": "stencil_ragged", "kind": "stencil", "ny": 1031, "nx": 777, "launches": 10,
         "seeded": 0, "words": 8, "map": "rowmajor"},
        # the headline stencil job: 4096 x 4096, 20 launches, 0.1 % of blocks racing
        {"name": "stencil_4096", "kind": "stencil", "ny": 4096, "nx": 4096,
         "launches": GRID_LAUNCHES, "seeded": 66, "words": 8, "map": "rowmajor"},
        # the same kernel with 4-byte shadow words, for programs whose data
        # leaves little memory for the checker
        {"name": "stencil_word4", "kind": "stencil", "ny": 2048, "nx": 3072,
         "launches": GRID_LAUNCHES, "seeded": 24, "words": 4, "map": "rowmajor"},
        # an ordinary graph, every access monitored (labels and the CSR arrays)
        {"name": "labelprop_csr", "kind": "labelprop", "vertices": 100003, "edges": 800024,
         "tpb": 256, "p_seed": 0.0, "csr": True},
        # the large graph: R-MAT of 2^22 vertices and 2^25 edges, 1 % of the
        # edges racing; the flagged set is large as well
        {"name": "labelprop_rmat22", "kind": "labelprop", "vertices": 1 << 22, "edges": 1 << 25,
         "tpb": 256, "p_seed": 0.01, "csr": False},
        # a user's own kernel rewritten by the source instrumenter: data-
        # dependent atomics through the general hook
        {"name": "user_histogram", "kind": "histogram", "n": 1500000, "bins": 4096, "plain": False},
        # an access program replayed by the interpreter: all kinds, spaces and
        # barrier scopes
        {"name": "access_program", "kind": "program", "blocks": 96, "threads": 256, "phases": 8,
         "words": 65536, "lds": 1024, "grouping": False},
        # many small jobs of all patterns in one persistent launch
        {"name": "batch_mixed", "kind": "batch", "jobs": 56, "mix": 3, "variant": 0, "order": 0,
         "map": "rowmajor"},
        # a burst of jobs handed to the serving loop, one large stencil among them
        {"name": "serve_burst", "kind": "serve", "jobs": 48, "mix": 4, "big": 2048},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["reduce", "job", "stencil", "stencil", "labelprop", "labelprop",
                       "histogram", "program", "batch", "serve"])
    if kind == "reduce":
        t = 64 * rng.randint(1, 16)
        n = 1 << rng.randint(1, (2 * t).bit_length() - 1)
        steps = n.bit_length() - 1
        # a step inside one wave: the sums stay defined, the race is found
        inside = [k for k in range(steps) if n >> (k + 1) <= 64]
        return {"kind": kind, "n": n, "threads": t, "blocks": _log(rng, 1, 2048),
                "drop": rng.choice(inside) if rng.random() < 0.3 else -1}
    if kind == "job":
        return {"kind": kind, "pattern": rng.choice(["reduce", "jacobi", "labelprop"]),
                "blocks": _log(rng, 1, 256), "threads": 64 * rng.randint(1, 16),
                "seeded": rng.random() < 0.3, "static": rng.random() < 0.4}
    if kind == "stencil":
        ny, nx = _log(rng, 16, 4096), _log(rng, 16, 4096)
        words = rng.choice([8, 8, 4])
        return {"kind": kind, "ny": ny, "nx": nx, "launches": rng.randint(1, GRID_LAUNCHES),
                "seeded": _log(rng, 1, 66) if rng.random() < 0.4 else 0, "words": words,
                "map": rng.choice(["rowmajor", "rowmajor", "4x4", "8x2"])}
    if kind == "labelprop":
        v = _log(rng, 200, 1 << 20)
        return {"kind": kind, "vertices": v, "edges": v * rng.randint(3, 12) + rng.randint(0, 7),
                "tpb": rng.choice([64, 128, 256, 512, 1024]),
                "p_seed": rng.choice([0.0, 0.01]), "csr": rng.random() < 0.4}
    if kind == "histogram":
        if rng.random() < 0.3:
            n = _log(rng, 1000, 100000)
            return {"kind": kind, "n": n, "bins": n // rng.randint(1, 4), "plain": True}
        return {"kind": kind, "n": _log(rng, 1000, 4000000), "bins": _log(rng, 32, 65536),
                "plain": False}
    if kind == "program":
        b, t, p = _log(rng, 4, 128), rng.randint(32, 512), rng.randint(1, 10)
        return {"kind": kind, "blocks": b, "threads": t, "phases": p,
                "words": min(1 << 20, b * t * p // rng.randint(1, 6)),
                "lds": _log(rng, 16, 4096), "grouping": rng.random() < 0.3}
    if kind == "batch":
        return {"kind": kind, "jobs": rng.randint(8, 56), "mix": rng.randint(0, 9999),
                "variant": rng.randint(0, 1),
                "order": rng.randint(0, 1), "map": rng.choice(sorted(MAPS))}
    return {"kind": "serve", "jobs": rng.randint(8, 56), "mix": rng.randint(0, 9999),
            "big": rng.choice([0, 1024, 2048])}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _grid(ny, nx, seed):
    return torch.rand((ny, nx), generator=_gen(seed), device="cuda", dtype=torch.float32)


def _ints(n, hi, seed):
    return torch.randint(0, hi, (n,), generator=_gen(seed), device="cuda", dtype=torch.int32)


def _seed_table(ny, nx, count, seed):
    if not count:
        return None
    rows = si.jacobi_seeds(ny, nx, int(seed), count=int(count))
    return torch.from_numpy(si.jacobi_seed_table(ny, nx, rows)).cuda() if len(rows) else None


def _graph(vertices, edges, p_seed, seed):
    """R-MAT edges folded into the vertices, in CSR, with the racing edges' mask."""
    g = _gen(seed)
    a, b, c = RMAT
    src = torch.zeros(edges, dtype=torch.int32, device="cuda")
    dst = torch.zeros_like(src)
    scale = max(1, (vertices - 1).bit_length())
    for level in range(scale):
        u = torch.rand(edges, generator=g, device="cuda")
        sbit = (u >= a + b).to(torch.int32)
        dbit = (((u >= a) & (u < a + b)) | (u >= a + b + c)).to(torch.int32)
        src |= sbit << (scale - 1 - level)
        dst |= dbit << (scale - 1 - level)
    src %= vertices
    dst %= vertices
    src, order = torch.sort(src, stable=True)
    col = dst[order].contiguous()
    rp = torch.zeros(vertices + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(src.long(), minlength=vertices), 0).to(torch.int32)
    mask = (torch.rand(edges, generator=g, device="cuda") < p_seed).to(torch.uint8)
    return rp, col, mask


def _job(pattern, blocks, threads, seeded, seed):
    """One job as the executors take it: (instance, its tensors, its result or
    None where a race reaches it, the words of its two buffers, LDS words of
    a block)."""
    inst = hr.Instance()
    inst.drop = -1
    inst.region[0] = inst.region[1] = hr.NO_REGION
    lds = 0
    if pattern == "reduce":
        n = 1 << ((2 * threads).bit_length() - 1)
        t = [_ints(n * blocks, 1 << 20, seed),
             torch.zeros(blocks * threads, dtype=torch.int32, device="cuda")]
        inst.pattern, inst.phases, inst.n = hr.HR_PAT_REDUCE, 1, n
        inst.threads, inst.blocks = threads, blocks
        inst.drop = n.bit_length() - 4 if seeded else -1      # a step inside one wave
        result, words, lds = t[1], [t[0].numel(), t[1].numel()], n
    elif pattern == "jacobi":
        side = 16 * math.isqrt(max(0, blocks - 1)) + 16
        t = [_grid(side, side, seed), torch.zeros((side, side), device="cuda"),
             _seed_table(side, side, 1 if seeded else 0, seed)]
        inst.pattern, inst.phases, inst.n, inst.ny = hr.HR_PAT_JACOBI, GRID_LAUNCHES, side, side
        result, words = t[0] if not seeded else None, [side * side, side * side]
    else:
        v = blocks * threads
        rp, col, mask = _graph(v, 8 * v, 0.01 if seeded else 0.0, seed)
        t = [torch.arange(v, dtype=torch.int32, device="cuda"), rp, col, mask]
        inst.pattern, inst.phases, inst.n = hr.HR_PAT_LABELPROP, GRAPH_LAUNCHES, v
        inst.threads = threads
        result, words = None if seeded else t[0], [v, 0]
    for i, x in enumerate(t):
        inst.data[i] = None if x is None else x.data_ptr()
    return inst, t, result, words, (blocks, lds)


def _jobs(count, mix, seed):
    """`count` jobs of the mixed manifest `mix`: pattern uniform, blocks
    log-uniform in 1..512, threads log-uniform in 64..1024, a tenth of them
    racing; their inputs come from `seed`."""
    specs = si.batched_manifest(int(mix), n_instances=int(count))
    names = {si.PAT_REDUCE: "reduce", si.PAT_JACOBI: "jacobi", si.PAT_LABELPROP: "labelprop"}
    return [_job(names[s["pattern"]], s["blocks"], s["threads"], s["seeded"], int(seed) + 7 * i)
            for i, s in enumerate(specs)]


class _Where:
    """Places of the monitored words in one mask: global words by region,
    LDS words by (array id, block)."""

    def __init__(self, regions, lds=()):
        """regions: (id, words); lds: (array id, blocks, words of a block)."""
        ids = [r for r, _ in regions] + [a for a, _, _ in lds] + [0]
        self.g = np.zeros(max(ids) + 1, np.int64)
        self.l, self.lw = np.zeros_like(self.g), np.zeros_like(self.g)
        self.size = 0
        for r, w in regions:
            self.g[r] = self.size
            self.size += w
        for a, blocks, w in lds:
            self.l[a], self.lw[a] = self.size, w
            self.size += blocks * w
        self.out, self.last = np.zeros(self.size, np.uint8), np.zeros(0, np.int64)

    def mask(self, space, region, block, index):
        at = np.where(space == hr.HR_LDS,
                      self.l[region] + self.lw[region] * block.astype(np.int64),
                      self.g[region]) + index.astype(np.int64)
        self.out[self.last] = 0            # the mask is kept: a pass writes what it flags
        self.out[at] = 1
        self.last = at
        return self.out


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case, kind = case, case["kind"]
    if kind == "reduce":
        n, t, b = case["n"], case["threads"], case["blocks"]
        s.inp = _ints(n * b, 1 << 20, seed)
        s.out = torch.zeros(b * t, dtype=torch.int32, device="cuda")
        s.ctx = hr.Context()
        s.regs = [s.ctx.shadow_alloc(s.inp), s.ctx.shadow_alloc(s.out)]
        s.where = _Where([(s.regs[0], n * b), (s.regs[1], t * b)], [(0, b, n)])
    elif kind == "stencil":
        ny, nx = case["ny"], case["nx"]
        s.first = _grid(ny, nx, seed)
        s.u = [s.first.clone(), torch.zeros_like(s.first)]
        s.tab = _seed_table(ny, nx, case["seeded"], seed)
        s.ctx = hr.Context(word4=case["words"] == 4)
        s.regs = [s.ctx.shadow_alloc(x, tile=MAPS[case["map"]]) for x in s.u]
        s.where = _Where([(r, ny * nx) for r in s.regs])
    elif kind == "labelprop":
        s.rp, s.col, s.mask = _graph(case["vertices"], case["edges"], case["p_seed"], seed)
        s.first = torch.arange(case["vertices"], dtype=torch.int32, device="cuda")
        s.label = s.first.clone()
        s.ctx = hr.Context(ring_capacity=1 << 21)
        s.r_label = s.ctx.shadow_alloc(s.label)
        s.kw = {}
        if case["csr"]:
            s.kw = {"r_row_ptr": s.ctx.shadow_alloc(s.rp), "r_col": s.ctx.shadow_alloc(s.col)}
        s.where = _Where([(s.r_label, case["vertices"])] + [
            (r, x.numel()) for r, x in zip(s.kw.values(), (s.rp, s.col))])
    elif kind == "histogram":
        s.keys = _ints(case["n"], case["bins"], seed)
        s.bins = torch.zeros(case["bins"], dtype=torch.int32, device="cuda")
        s.ctx = hr.Context()
        s.regs = [s.ctx.shadow_alloc(s.keys), s.ctx.shadow_alloc(s.bins)]
        s.where = _Where([(s.regs[0], case["n"]), (s.regs[1], case["bins"])])
    elif kind == "program":
        p = si.random_program(int(seed), launches=2, blocks=case["blocks"],
                              threads=case["threads"], phases=case["phases"], max_ops=4,
                              global_regions=2, global_words=case["words"],
                              lds_words=case["lds"], kind_p=(0.94, 0.02, 0.04))
        s.progs = [hr.DeviceProgram(launch) for launch in p.launches]
        s.data = [torch.zeros(w, dtype=torch.int32, device="cuda") for w in p.global_words]
        s.lds = p.lds_words
        s.ctx = hr.Context(ring_capacity=1 << 18, wave_grouping=case["grouping"])
        s.regs = [s.ctx.shadow_alloc(x) for x in s.data]
        s.where = _Where([(r, case["words"]) for r in s.regs],
                         [(0, case["blocks"], case["lds"])])
    elif kind == "job":
        s.job = _job(case["pattern"], case["blocks"], case["threads"], case["seeded"], seed)
        s.where = _where_jobs([s.job])
    elif kind == "batch":
        s.jobs = _jobs(case["jobs"], case["mix"], seed)
        s.ctx = hr.Context(ring_capacity=1 << 20)
        s.batch = hr.Batch(s.ctx, [j[0] for j in s.jobs])
        regs = [s.batch.regions(i) for i in range(len(s.jobs))]
        s.where = _Where([(r, w) for rs, j in zip(regs, s.jobs) for r, w in zip(rs, j[3])
                          if r != hr.NO_REGION],
                         [(rs[0], *j[4]) for rs, j in zip(regs, s.jobs)])
    else:
        s.jobs = _jobs(case["jobs"], case["mix"], seed)
        if case["big"]:
            blocks = (case["big"] // 16) ** 2
            s.jobs.insert(len(s.jobs) // 2, _job("jacobi", blocks, 256, True, seed))
        s.ctx = hr.Context(ring_capacity=1 << 20)
        s.arrivals = np.zeros(len(s.jobs))
        s.where = _where_jobs(s.jobs)
    return s


def _where_jobs(jobs):
    """Job j's buffers as regions 2j and 2j + 1, its LDS as array 2j."""
    return _Where([(2 * i + k, w) for i, j in enumerate(jobs) for k, w in enumerate(j[3])],
                  [(2 * i, *j[4]) for i, j in enumerate(jobs)])


# ------------------------------------------------------------------ one pass
def _report(s):
    recs, status = s.ctx.report()
    return {"flagged": s.where.mask(recs["space"], recs["region"], recs["block"], recs["index"]),
            "status": status}


def _flagged(where, sets):
    """The mask of per-job key sets (space, region 0 or 1, block if LDS, index)."""
    rows = np.array([(sp, 2 * j + rg, b, i) for j, keys in enumerate(sets)
                     for sp, rg, b, i in keys], dtype=np.int64).reshape(-1, 4)
    return where.mask(*rows.T)


def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "reduce":
        s.ctx.reset()
        s.ctx.reduce_check(s.regs[0], s.regs[1], s.inp, s.out, drop=case["drop"], n=case["n"],
                           threads=case["threads"], blocks=case["blocks"])
        s.ctx.kernel_end()
        return dict(_report(s), out=s.out)
    if kind == "stencil":
        s.ctx.reset()
        s.u[0].copy_(s.first)
        for k in range(case["launches"]):
            a, b = k % 2, 1 - k % 2
            s.ctx.jacobi_check(s.regs[a], s.regs[b], s.u[a], s.u[b], s.tab)
            s.ctx.kernel_end()
        got = _report(s)
        if not case["seeded"]:
            got["grid"] = s.u[case["launches"] % 2]
        return got
    if kind == "labelprop":
        s.ctx.reset()
        s.label.copy_(s.first)
        for _ in range(GRAPH_LAUNCHES):
            s.ctx.labelprop_check(s.r_label, s.label, s.rp, s.col, s.mask, tpb=case["tpb"], **s.kw)
            s.ctx.kernel_end()
        got = _report(s)
        if not case["p_seed"]:
            got["label"] = s.label          # ten sweeps reach the fixed point
        return got
    if kind == "histogram":
        s.ctx.reset()
        s.bins.zero_()
        examples.launch("histogram", s.ctx, s.regs, ((case["n"] + 255) // 256,), (256,), s.keys,
                        s.bins, case["n"], int(case["plain"]))
        s.ctx.kernel_end()
        got = _report(s)
        if not case["plain"]:
            got["bins"] = s.bins
        return got
    if kind == "program":
        s.ctx.reset()
        for p in s.progs:
            s.ctx.program_check(p, s.regs, s.lds)
            s.ctx.kernel_end()
        return _report(s)
    if kind == "job":
        keys, status = hr.job_run(s.job[0], static=case["static"])
        got = {"flagged": _flagged(s.where, [keys]), "status": status}
        if s.job[2] is not None:
            got["result"] = s.job[2]
        return got
    if kind == "batch":
        s.ctx.reset()
        s.batch.run(variant=case["variant"], order=case["order"], tile=MAPS[case["map"]])
        got = _report(s)
        got["results"] = [j[2] for j in s.jobs if j[2] is not None]
        return got
    sets, times = hr.serve(s.ctx, [j[0] for j in s.jobs], s.arrivals)
    return {"flagged": _flagged(s.where, sets), "counts": np.array([t.flagged for t in times]),
            "status": np.array([t.status for t in times]),
            "results": [j[2] for j in s.jobs if j[2] is not None]}


# ------------------------------------------------------------------ the floor
def _job_work(pattern, blocks, threads):
    """(bytes, operations) of one job: its data and its shadow words."""
    if pattern == "reduce":
        n = 1 << ((2 * threads).bit_length() - 1)
        return blocks * (n * (4 + 16) + threads * (4 + 16)), blocks * n
    if pattern == "jacobi":
        cells = (16 * math.isqrt(max(0, blocks - 1)) + 16) ** 2
        return GRID_LAUNCHES * cells * (8 + 32), GRID_LAUNCHES * cells * 5
    v = blocks * threads
    return GRAPH_LAUNCHES * (v * (4 + 8 + 16) + 8 * v * 5), GRAPH_LAUNCHES * 8 * v


def _mean_job_work(count):
    # the manifest's mean: a third of each pattern, 82 blocks and 346 threads
    each = [_job_work(p, 82, 346) for p in ("reduce", "jacobi", "labelprop")]
    return [count * sum(e[i] for e in each) / 3 for i in (0, 1)]


def work(case):
    """Bytes: the program's data, and its shadow words read and written once
    per launch.  Operations: the program's own."""
    kind = case["kind"]
    if kind == "reduce":
        n, t, b = case["n"], case["threads"], case["blocks"]
        return {"bytes": b * (n + t) * (4 + 16), "flops": b * n}
    if kind == "stencil":
        cells = case["ny"] * case["nx"] * case["launches"]
        return {"bytes": cells * (8 + 4 * case["words"]), "flops": cells * 5}
    if kind == "labelprop":
        v, e = case["vertices"], case["edges"]
        each = v * (4 + 8 + 16) + e * (4 + 1)
        if case["csr"]:
            each += 16 * (v + e)
        return {"bytes": GRAPH_LAUNCHES * each, "flops": GRAPH_LAUNCHES * e}
    if kind == "histogram":
        return {"bytes": (case["n"] + case["bins"]) * (4 + 16), "flops": case["n"]}
    if kind == "program":
        ops = 2 * 2 * case["blocks"] * case["threads"] * case["phases"]
        return {"bytes": ops * (4 + 4) + 2 * 2 * case["words"] * 16, "flops": ops}
    if kind == "job":
        b, f = _job_work(case["pattern"], case["blocks"], case["threads"])
        return {"bytes": b, "flops": f}
    b, f = _mean_job_work(case["jobs"])
    if case.get("big"):
        more = _job_work("jacobi", (case["big"] // 16) ** 2, 256)
        b, f = b + more[0], f + more[1]
    return {"bytes": b, "flops": f}


def _sweeps(u, launches):
    """The 5-point sweep in 64 bits; a neighbour outside the grid is the cell itself."""
    u = u.double()
    for _ in range(launches):
        n = torch.cat([u[:1], u[:-1]], 0)
        so = torch.cat([u[1:], u[-1:]], 0)
        w = torch.cat([u[:, :1], u[:, :-1]], 1)
        e = torch.cat([u[:, 1:], u[:, -1:]], 1)
        u = 0.2 * (u + n + so + w + e)
    return u


def exact(case, seed):
    """The race-free stencil's grid is the only output in floating point."""
    if case["kind"] != "stencil" or case["seeded"]:
        return None
    return {"flagged": None, "status": None,
            "grid": _sweeps(_grid(case["ny"], case["nx"], seed), case["launches"])}
