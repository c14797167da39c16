"""Label propagation cut into equal pieces of vertices and edges: hubs whose
edges span pieces, pieces without a vertex or without an edge, and pieces of
more vertices than a block loads at a time, through every path that cuts
(a context's launch, the static scratch, a batch, the serving loop) and
beside another stream."""
import numpy as np
import pytest

from oracle import closed_forms as cf

pytestmark = pytest.mark.gpu


def graph(name):
    rng = np.random.default_rng(21)
    n = {"under": 2047, "over": 2049, "tall": 4300000}.get(name, 2500)
    deg = np.zeros(n, np.int64)
    if name in ("under", "over"):
        deg[:] = rng.integers(0, 12, n)
    elif name == "first_hub":
        deg[:] = 1
        deg[0] = 30000
    elif name == "last_hub":
        deg[::3] = 2
        deg[-1] = 20001
    elif name == "only_hub":
        deg[1234] = 50000
    elif name == "two_hubs":
        deg[:] = rng.integers(0, 3, n)
        deg[700], deg[701] = 9000, 9001
    elif name == "tall":                     # above 1,024 vertices a piece
        deg[rng.integers(0, n, 3000)] = 1
        deg[17], deg[n - 5] = 5000, 3000
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = rng.integers(0, n, max(1, int(rp[-1]))).astype(np.int32)
    return rp, col


def fixed_point(rp, col):
    n = rp.shape[0] - 1
    src, col = np.repeat(np.arange(n), np.diff(rp)), col[:rp[-1]]
    want = np.arange(n, dtype=np.int32)
    while True:
        nxt = want.copy()
        np.minimum.at(nxt, col, want[src])
        if (nxt == want).all():
            return want
        want = nxt


NAMES = ["under", "over", "first_hub", "last_hub", "only_hub", "two_hubs", "no_edges", "tall"]


@pytest.mark.parametrize("name", NAMES)
def test_context(name):
    import torch
    from paper_2401_04701_amd import hr
    rp, col = graph(name)
    n, m = rp.shape[0] - 1, int(rp[-1])
    mask = (np.random.default_rng(12).random(col.shape[0]) < 0.02).astype(np.uint8)
    print("[case] pieces", name, flush=True)
    up = lambda a: torch.from_numpy(a).cuda()
    rp_d, col_d, mask_d, none = up(rp), up(col), up(mask), up(np.zeros_like(mask))
    label = torch.arange(n, dtype=torch.int32, device="cuda")
    with hr.Context(count_checks=True, ring_capacity=1 << 18) as ctx:
        regs = [ctx.shadow_alloc(label), ctx.shadow_alloc(rp_d), ctx.shadow_alloc(col_d)]
        for L in range(2):
            ctx.labelprop_check(regs[0], label, rp_d, col_d, mask_d, tpb=192, r_row_ptr=regs[1],
                                r_col=regs[2])
            ctx.kernel_end()
        assert ctx.check_count() == 2 * (3 * n + 2 * m + int(mask[:m].sum()))
        assert ctx.flagged() == cf.labelprop_flagged(rp, col[:m], mask[:m]) and ctx.status == 0
        ctx.reset()
        label.copy_(torch.arange(n, dtype=torch.int32, device="cuda"))
        for _ in range(40):
            ctx.labelprop_check(regs[0], label, rp_d, col_d, none, tpb=192)
            ctx.kernel_end()
        assert ctx.flagged() == set()
    assert (label.cpu().numpy() == fixed_point(rp, col)).all()


def instance(hr, rp, col, mask, threads):
    """(instance, its tensors)."""
    import torch
    up = lambda a: torch.from_numpy(a).cuda()
    t = [torch.arange(rp.shape[0] - 1, dtype=torch.int32, device="cuda"), up(rp), up(col),
         up(mask)]
    inst = hr.Instance()
    inst.drop = -1
    inst.region[0] = inst.region[1] = hr.NO_REGION
    inst.pattern, inst.phases, inst.n = hr.HR_PAT_LABELPROP, 40, rp.shape[0] - 1
    inst.threads = threads
    for i, x in enumerate(t):
        inst.data[i] = x.data_ptr()
    return inst, t


@pytest.mark.parametrize("path", ["static", "batch", "serve"])
def test_executors(path):
    """All graphs as jobs, seeded and not: flagged sets, and the labels of the
    jobs without races after 40 phases."""
    import torch
    from paper_2401_04701_amd import hr
    print("[case] pieces", path, flush=True)
    graphs = [graph(x) for x in NAMES if x != "tall"]
    masks = [(np.random.default_rng(i).random(g[1].shape[0]) < 0.02 * (i % 2)).astype(np.uint8)
             for i, g in enumerate(graphs)]
    want = [{k for k in cf.labelprop_flagged(rp, col[:rp[-1]], m[:rp[-1]])}
            for (rp, col), m in zip(graphs, masks)]
    jobs = [instance(hr, *g, m, 64 if i % 3 else 320)
            for i, (g, m) in enumerate(zip(graphs, masks))]
    if path == "static":
        got = [hr.job_run(j[0], static=True)[0] for j in jobs]
    elif path == "serve":
        with hr.Context(ring_capacity=1 << 18) as ctx:
            got, _ = hr.serve(ctx, [j[0] for j in jobs], np.zeros(len(jobs)))
    else:
        with hr.Context(ring_capacity=1 << 18) as ctx:
            with hr.Batch(ctx, [j[0] for j in jobs]) as b:
                for variant in (0, 1):
                    for j in jobs:
                        j[1][0].copy_(torch.arange(j[0].n, dtype=torch.int32, device="cuda"))
                    ctx.reset()
                    b.run(variant=variant)
                    got = b.split(ctx.flagged())
                    assert [set(g) for g in got] == want
    assert [set(g) for g in got] == want
    for (rp, col), m, j in zip(graphs, masks, jobs):
        if not m.any():
            assert (j[1][0].cpu().numpy() == fixed_point(rp, col)).all()


@pytest.mark.parametrize("capture", [False, True])
def test_two_streams_and_capture(capture):
    """Jobs of one context on two streams share its room for pieces; a captured
    launch does not use it."""
    import torch
    from paper_2401_04701_amd import hr
    print("[case] pieces capture", capture, flush=True)
    graphs = [graph("two_hubs"), graph("first_hub")]
    up = lambda a: torch.from_numpy(a).cuda()
    dev = [[up(a) for a in (*g, np.zeros(g[1].shape[0], np.uint8))] for g in graphs]
    labels = [torch.arange(g[0].shape[0] - 1, dtype=torch.int32, device="cuda") for g in graphs]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    with hr.Context() as ctx:
        regs = [ctx.shadow_alloc(x) for x in labels]
        torch.cuda.synchronize()
        if capture:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                for i in range(2):
                    ctx.labelprop_check(regs[i], labels[i], *dev[i])
            for _ in range(20):
                ctx.reset()
                g.replay()
                assert ctx.flagged() == set()
        else:
            for _ in range(40):
                for i in range(2):
                    with torch.cuda.stream(streams[i]):
                        ctx.labelprop_check(regs[i], labels[i], *dev[i])
                ctx.kernel_end()
            torch.cuda.synchronize()
            assert ctx.flagged() == set()
    for (rp, col), x in zip(graphs, labels):
        assert (x.cpu().numpy() == fixed_point(rp, col)).all()


def test_jobs_on_alternating_streams():
    """One context's jobs on two streams in turn, each job its own graph."""
    import torch
    from paper_2401_04701_amd import hr
    print("[case] pieces alternating streams", flush=True)
    graphs = [graph("two_hubs"), graph("first_hub")]
    up = lambda a: torch.from_numpy(a).cuda()
    dev = [[up(a) for a in (*g, np.zeros(g[1].shape[0], np.uint8))] for g in graphs]
    labels = [torch.arange(g[0].shape[0] - 1, dtype=torch.int32, device="cuda") for g in graphs]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    with hr.Context() as ctx:
        regs = [ctx.shadow_alloc(x) for x in labels]
        torch.cuda.synchronize()
        for job in range(8):
            i = job % 2
            with torch.cuda.stream(streams[i]):
                ctx.reset()
                for _ in range(10):
                    ctx.labelprop_check(regs[i], labels[i], *dev[i])
                    ctx.kernel_end()
                assert ctx.flagged() == set()
    for (rp, col), x in zip(graphs, labels):
        assert (x.cpu().numpy() == fixed_point(rp, col)).all()
