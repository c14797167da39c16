"""Every halo read of the stencil is in its cell's word.  The owner applies it
from the grid's geometry, apart from the load itself, so a read that is left out
there would not show in the sweep's own flagged set.  Here a second kernel of the
same epoch writes every cell as the cell's own block and thread, at the same
clocks: such a write races with the other blocks' reads of the cell and with
nothing else, so the flagged cells are those that another block read."""
import numpy as np
import pytest

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu


def owners_write(ny, nx):
    """One launch: thread t of block b writes the old grid's cell that it owns."""
    nby, nbx = (ny + 15) // 16, (nx + 15) // 16
    b, t = np.divmod(np.arange(nby * nbx * 256), 256)
    y, x = b // nbx * 16 + t // 16, b % nbx * 16 + t % 16
    inside = (y < ny) & (x < nx)
    return si.Launch(blocks=nby * nbx, threads=256, scope=np.zeros(1, np.uint8),
                     wave_mask=np.zeros(1, np.uint64),
                     op_off=np.concatenate([[0], np.cumsum(inside)]).astype(np.int32),
                     ops=((y * nx + x)[inside] | 1 << 27).astype(np.uint32))


@pytest.mark.parametrize("how", ["exclusive", "shared", "in front"])
@pytest.mark.parametrize("kind", ["plain", "word4", "tiled", "table", "narrow"])
@pytest.mark.parametrize("ny,nx", [(16, 16), (1, 33), (33, 1), (48, 64), (50, 37)])
def test_cells_read_by_other_blocks(ny, nx, kind, how):
    import torch
    from paper_2401_04701_amd import hr
    print("[case] owner reads", ny, nx, kind, how, flush=True)
    launch = owners_write(ny, nx)
    want = oracle.flagged(np.concatenate([oracle.model_jacobi(ny, nx, 1, None),
                                          oracle.model_launch(launch, 0)]))
    y, x = np.indices((ny, nx))
    edge = ((y % 16 == 0) & (y > 0)) | ((y % 16 == 15) & (y + 1 < ny)) | \
           ((x % 16 == 0) & (x > 0)) | ((x % 16 == 15) & (x + 1 < nx))
    assert {k[3] for k in want} == set(np.nonzero(edge.ravel())[0].tolist())
    prog = hr.DeviceProgram(launch)
    u = [torch.rand((ny, nx), device="cuda"), torch.zeros((ny, nx), device="cuda")]
    kw = {"word4": {"word4": True}, "table": {"fsm_table": True},
          "narrow": {"wave_bits": 3}}.get(kind, {})
    with hr.Context(**kw) as ctx:
        regs = [ctx.shadow_alloc(a, tile=(2, 2) if kind == "tiled" else None) for a in u]
        other = torch.cuda.Stream()
        torch.cuda.synchronize()
        stream = other if how == "shared" else None
        if how != "exclusive":
            ctx.program_check(prog, regs, 0)
        if how == "shared":
            torch.cuda.synchronize()
        ctx.jacobi_check(regs[0], regs[1], u[0], u[1], None, stream=stream)
        if how == "exclusive":
            ctx.program_check(prog, regs, 0)
        torch.cuda.synchronize()
        got = {(0, regs.index(k[1]), 0, k[3]) for k in ctx.flagged()}
        assert ctx.status == 0
    assert got == want
