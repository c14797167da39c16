"""Owner updates in the stencil: one thread applies every access to a word.
Grids at the tiles' edges with seeds on every side, in-place sweeps, and
launch epochs shared with another kernel (before or after the sweep, on its
stream or another one, or captured), against the oracle."""
import numpy as np
import pytest

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2401_04701_amd import hr
    torch.cuda.set_device(0)
    return torch, hr


def say(*a):
    print("[case]", *a, flush=True)


def full_table(ny, nx):
    """Every block seeded that has a neighbour cell to write."""
    nb = ((ny + 15) // 16) * ((nx + 15) // 16)
    return si.jacobi_seed_table(ny, nx, si.jacobi_seeds(ny, nx, 5, count=nb))


def keys_of(ctx, regs):
    m = {r: i for i, r in enumerate(regs)}
    return {(s, m[r] if s == 0 else r, b, i) for s, r, b, i in ctx.flagged()}


@pytest.mark.parametrize("word4", [False, True])
@pytest.mark.parametrize("wave_bits", [6, 3])
@pytest.mark.parametrize("ny,nx", [(1, 1), (1, 33), (17, 1), (16, 16), (31, 32), (33, 47),
                                   (48, 64), (65, 17)])
def test_edges_seeded_on_every_side(env, ny, nx, wave_bits, word4):
    torch, hr = env
    say("owner edges", ny, nx, "wave_bits", wave_bits, "word4", word4)
    tab = full_table(ny, nx)
    u = [torch.from_numpy(si.jacobi_grid(ny, nx, 3)).cuda(),
         torch.zeros((ny, nx), device="cuda")]
    with hr.Context(wave_bits=wave_bits, word4=word4, count_checks=True) as ctx:
        regs = [ctx.shadow_alloc(x) for x in u]
        for L in range(3):
            ctx.jacobi_check(regs[L % 2], regs[1 - L % 2], u[L % 2], u[1 - L % 2],
                             torch.from_numpy(tab).cuda() if L != 1 else None)
            ctx.kernel_end()
        got, st, n = keys_of(ctx, regs), ctx.status, ctx.check_count()
    log = np.concatenate([oracle.model_jacobi(ny, nx, 1, tab if L != 1 else None, launch0=L)
                          for L in range(3)])
    assert st == 0 and n == len(log)
    assert got == oracle.flagged(log.copy(), 1 << wave_bits)


@pytest.mark.parametrize("word4", [False, True])
def test_in_place(env, word4):
    """One region as both grids: the halo reads race with the owners' writes."""
    torch, hr = env
    ny, nx = 40, 50
    say("in place word4", word4)
    u = torch.from_numpy(si.jacobi_grid(ny, nx, 3)).cuda()
    with hr.Context(word4=word4) as ctx:
        r = ctx.shadow_alloc(u)
        ctx.jacobi_check(r, r, u, u, None)
        ctx.kernel_end()
        got = keys_of(ctx, [r])
    log = oracle.model_jacobi(ny, nx, 1, None)
    log["region"][log["space"] == 0] = 0
    assert got == oracle.flagged(log) and got


def writes_by(block, cells, region):
    """One launch in which only `block` acts: its threads write the cells."""
    threads = 64
    off = np.zeros((block + 1) * threads + 1, np.int32)
    per = -(-len(cells) // threads)
    ops = []
    for t in range(threads):
        ops += [c | region << 24 | 1 << 27 for c in cells[t * per:(t + 1) * per]]
        off[block * threads + t + 1] = len(ops)
    return si.Launch(blocks=block + 1, threads=threads, scope=np.zeros(1, np.uint8),
                     wave_mask=np.zeros(1, np.uint64), op_off=off,
                     ops=np.array(ops, np.uint32))


@pytest.mark.parametrize("word4", [False, True])
@pytest.mark.parametrize("where", ["same", "other", "captured"])
@pytest.mark.parametrize("first", ["sweep", "writes"])
@pytest.mark.parametrize("region", [0, 1])
def test_epoch_shared_with_another_kernel(env, region, first, where, word4):
    """A kernel that writes cells of one grid in the sweep's launch epoch:
    every cell it writes races with the sweep, whichever runs first."""
    torch, hr = env
    ny, nx = 33, 40
    cells = list(range(0, ny * nx, 7))
    launch = writes_by(9, cells, region)
    say("shared epoch", region, first, where, "word4", word4)
    u = [torch.from_numpy(si.jacobi_grid(ny, nx, 3)).cuda(),
         torch.zeros((ny, nx), device="cuda")]
    prog = hr.DeviceProgram(launch)
    log = np.concatenate([oracle.model_jacobi(ny, nx, 1, None), oracle.model_launch(launch, 0)])
    want = oracle.flagged(log)
    assert {k[3] for k in want} == set(cells)
    with hr.Context(word4=word4) as ctx:
        regs = [ctx.shadow_alloc(x) for x in u]
        other = torch.cuda.Stream()

        def sweep():
            ctx.jacobi_check(regs[0], regs[1], u[0], u[1], None)

        def writes():
            if where != "other":
                return ctx.program_check(prog, regs, 0)
            with torch.cuda.stream(other):
                ctx.program_check(prog, regs, 0)

        def job():
            for f in ([sweep, writes] if first == "sweep" else [writes, sweep]):
                f()

        if where != "captured":
            torch.cuda.synchronize()
            job()
            torch.cuda.synchronize()
            ctx.kernel_end()
            assert keys_of(ctx, regs) == want
            return
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            job()
        for _ in range(3):
            ctx.reset()
            g.replay()
            assert keys_of(ctx, regs) == want


@pytest.mark.parametrize("recorded", ["sweep", "writes"])
@pytest.mark.parametrize("order", ["eager first", "graph first"])
@pytest.mark.parametrize("where", ["same", "other"])
def test_epoch_shared_with_a_graph(env, where, order, recorded):
    """One epoch's sweep and writes, one launched and one recorded (on the same
    stream or another one) and then replayed on a third, whichever is first."""
    torch, hr = env
    ny, nx = 33, 40
    cells = list(range(0, ny * nx, 7))
    launch = writes_by(9, cells, 1)
    say("epoch and graph", where, order, recorded)
    u = [torch.from_numpy(si.jacobi_grid(ny, nx, 3)).cuda(),
         torch.zeros((ny, nx), device="cuda")]
    prog = hr.DeviceProgram(launch)
    want = oracle.flagged(np.concatenate([oracle.model_jacobi(ny, nx, 1, None),
                                          oracle.model_launch(launch, 0)]))
    streams = [torch.cuda.Stream() for _ in range(3)]
    with hr.Context() as ctx:
        regs = [ctx.shadow_alloc(x) for x in u]
        calls = [lambda: ctx.jacobi_check(regs[0], regs[1], u[0], u[1], None),
                 lambda: ctx.program_check(prog, regs, 0)]
        if recorded == "sweep":
            calls.reverse()
        eager, graph = calls
        torch.cuda.synchronize()

        def launch_eager():
            with torch.cuda.stream(streams[0]):
                eager()

        g = torch.cuda.CUDAGraph()
        if order == "eager first":
            launch_eager()
        with torch.cuda.graph(g, stream=streams[0 if where == "same" else 1]):
            graph()
        if order == "graph first":
            launch_eager()
        for _ in range(3):
            with torch.cuda.stream(streams[2]):
                g.replay()
        torch.cuda.synchronize()
        ctx.kernel_end()
        assert keys_of(ctx, regs) == want


@pytest.mark.parametrize("word4", [False, True])
@pytest.mark.parametrize("ny,nx", [(16, 4095), (17, 4096), (16 * 15, 16 * 17 + 1), (270, 300)])
def test_tiles_over_the_dies(env, ny, nx, word4):
    """Grids of 255, 256, 512 and other counts of tiles: the blocks' order over
    the chip's dies covers every tile once."""
    torch, hr = env
    say("tiles over dies", ny, nx, "word4", word4)
    seeds = si.jacobi_seeds(ny, nx, 8, count=40)
    tab = torch.from_numpy(si.jacobi_seed_table(ny, nx, seeds)).cuda()
    u = [torch.from_numpy(si.jacobi_grid(ny, nx, 3)).cuda(),
         torch.zeros((ny, nx), device="cuda")]
    first = u[0].clone()
    with hr.Context(word4=word4, count_checks=True) as ctx:
        regs = [ctx.shadow_alloc(x) for x in u]
        ctx.jacobi_check(regs[0], regs[1], u[0], u[1], None)
        ctx.kernel_end()
        assert ctx.flagged() == set()
        want = torch.zeros_like(first)
        hr.jacobi_plain(first, want, None)
        assert torch.equal(u[1], want)
        x = first.double()
        n, s = torch.cat([x[:1], x[:-1]]), torch.cat([x[1:], x[-1:]])
        w, e = torch.cat([x[:, :1], x[:, :-1]], 1), torch.cat([x[:, 1:], x[:, -1:]], 1)
        assert (want.double() - 0.2 * (x + n + s + w + e)).abs().max() < 1e-6
        ctx.jacobi_check(regs[0], regs[1], u[0], u[1], tab)
        ctx.kernel_end()
        got, st = keys_of(ctx, regs), ctx.status
    assert st == 0 and got == {(0, 1, 0, k[3]) for k in oracle.flagged(
        oracle.model_jacobi(ny, nx, 1, tab.cpu().numpy()))}


@pytest.mark.parametrize("side", [33, 1100])       # below and above 4,096 records
def test_reports_do_not_share_memory(env, side):
    """A report's records stay as they were when the next report is made."""
    torch, hr = env
    say("two reports", side)
    tab = torch.from_numpy(full_table(side, side)).cuda()
    u = [torch.from_numpy(si.jacobi_grid(side, side, 3)).cuda(),
         torch.zeros((side, side), device="cuda")]
    with hr.Context() as ctx:
        regs = [ctx.shadow_alloc(x) for x in u]
        ctx.jacobi_check(regs[0], regs[1], u[0], u[1], tab)
        ctx.kernel_end()
        first = ctx.report()[0]
        kept = first.copy()
        assert (len(first) > 4096) == (side > 1000)
        ctx.reset()
        assert len(ctx.report()[0]) == 0
        again = ctx.report()[0]
        assert len(again) == 0 and (first == kept).all()
