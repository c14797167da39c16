"""Label propagation over a range of a larger graph's rows: row_ptr[0] > 0, with
the whole col and mask, so the edges below row_ptr[0] belong to no vertex.
Every path, below and above the vertex count from which a launch is cut into
pieces: labels, access counts and flagged sets are those of the range alone."""
import numpy as np
import pytest

from oracle import closed_forms as cf

pytestmark = pytest.mark.gpu

SIZES = [100, 2047, 2048, 2500, 40000]


def rows(n, before, seed, p_seed):
    """(row_ptr of n rows that begin at edge `before`, col, mask): the edges
    before them and 30 behind them target the rows' vertices as well."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 8, n)
    deg[0], deg[n // 2], deg[-1] = 0, 3000, 17
    rp = (before + np.concatenate([[0], np.cumsum(deg)])).astype(np.int32)
    col = rng.integers(0, n, int(rp[-1]) + 30).astype(np.int32)
    mask = (rng.random(col.shape[0]) < p_seed).astype(np.uint8)
    mask[:before:3] = 1
    return rp, col, mask


def own(rp, col, mask):
    """The rows' edges alone: (row_ptr, col, mask) with row_ptr[0] == 0."""
    a, b = int(rp[0]), int(rp[-1])
    return rp - rp[0], col[a:b], mask[a:b]


def fixed_point(rp, col):
    n = rp.shape[0] - 1
    src = np.repeat(np.arange(n), np.diff(rp))
    want = first_labels(n)
    while True:
        nxt = want.copy()
        np.minimum.at(nxt, col, want[src])
        if (nxt == want).all():
            return want
        want = nxt


def first_labels(n):
    return np.arange(5, n + 5, dtype=np.int32)     # above 0: a label 0 is a stranger's


def device(torch, *arrays):
    return [torch.from_numpy(a).cuda() for a in arrays]


@pytest.mark.parametrize("grouping", [False, True])
@pytest.mark.parametrize("n", SIZES)
def test_context(n, grouping):
    import torch
    from paper_2401_04701_amd import hr
    print("[case] slice", n, "grouping", grouping, flush=True)
    rp, col, mask = rows(n, 50, n, 0.02)
    orp, ocol, omask = own(rp, col, mask)
    m = ocol.shape[0]
    rp_d, col_d, mask_d, none = device(torch, rp, col, mask, np.zeros_like(mask))
    label = torch.from_numpy(first_labels(n)).cuda()
    with hr.Context(count_checks=True, ring_capacity=1 << 18, wave_grouping=grouping) as ctx:
        regs = [ctx.shadow_alloc(label), ctx.shadow_alloc(rp_d), ctx.shadow_alloc(col_d)]
        for _ in range(2):
            ctx.labelprop_check(regs[0], label, rp_d, col_d, mask_d, tpb=192, r_row_ptr=regs[1],
                                r_col=regs[2])
            ctx.kernel_end()
        assert ctx.check_count() == 2 * (3 * n + 2 * m + int(omask.sum()))
        assert ctx.flagged() == cf.labelprop_flagged(orp, ocol, omask) and ctx.status == 0
        ctx.reset()
        label.copy_(torch.from_numpy(first_labels(n)))
        for _ in range(40):
            ctx.labelprop_check(regs[0], label, rp_d, col_d, none, tpb=192)
            ctx.kernel_end()
        assert ctx.flagged() == set()
    assert (label.cpu().numpy() == fixed_point(orp, ocol)).all()
    plain = torch.from_numpy(first_labels(n)).cuda()
    for _ in range(40):
        hr.labelprop_plain(plain, rp_d, col_d, none, tpb=192)
    assert torch.equal(plain, label)


@pytest.mark.parametrize("path", ["job", "static", "serve", "batch"])
def test_executors(path):
    import torch
    from paper_2401_04701_amd import hr
    print("[case] slices", path, flush=True)
    graphs = [rows(n, before, i, 0.02 * (i % 2))
              for i, (n, before) in enumerate((n, b) for n in SIZES for b in (0, 1, 5000))]
    for i, g in enumerate(graphs):
        if i % 2 == 0:
            g[2][:] = 0
    jobs = []
    for i, (rp, col, mask) in enumerate(graphs):
        t = device(torch, first_labels(rp.shape[0] - 1), rp, col, mask)
        inst = hr.Instance()
        inst.drop = -1
        inst.region[0] = inst.region[1] = hr.NO_REGION
        inst.pattern, inst.phases, inst.n = hr.HR_PAT_LABELPROP, 40, rp.shape[0] - 1
        inst.threads = 64 if i % 3 else 320
        for k, x in enumerate(t):
            inst.data[k] = x.data_ptr()
        jobs.append((inst, t))
    instances = [j[0] for j in jobs]
    if path in ("job", "static"):
        got = [hr.job_run(i, static=path == "static")[0] for i in instances]
    else:
        with hr.Context(ring_capacity=1 << 18) as ctx:
            if path == "serve":
                got, _ = hr.serve(ctx, instances, np.zeros(len(jobs)))
            else:
                with hr.Batch(ctx, instances) as b:
                    b.run()
                    got = b.split(ctx.flagged())
                    assert ctx.status == 0
    for g, (_, t), found in zip(graphs, jobs, got):
        orp, ocol, omask = own(*g)
        assert set(found) == cf.labelprop_flagged(orp, ocol, omask)
        if not omask.any():
            assert (t[0].cpu().numpy() == fixed_point(orp, ocol)).all()
