"""Label propagation where a block's lanes share its vertices' edges: the
flagged set, the number of checked accesses and the labels, at the edges of
the mapping (vertices per block, edges per round of lanes, empty rows, hubs,
logical blocks that straddle hardware blocks)."""
import numpy as np
import pytest

import oracle
from oracle import closed_forms as cf

pytestmark = pytest.mark.gpu


def graph(name):
    """(row_ptr, col): degrees chosen at the mapping's edges."""
    rng = np.random.default_rng(11)
    deg = {
        "one": [3],
        "block_less_one": [2] * 31,
        "block_exact": [1] * 32,
        "block_plus_one": [0] * 32 + [5],
        "round_less_one": [1023] + [0] * 40,
        "round_exact": [0, 1024, 0, 0],
        "round_plus_one": [0] * 31 + [1025, 1, 0, 2],
        "empty_rows": [0, 0, 7, 0, 0, 0, 9, 0] * 24,
        "two_hubs": [2500] + [1] * 30 + [3000] + [2] * 100,
        # above 131,072 vertices a block takes 64, above 262,144 more
        "wide": list(rng.integers(0, 3, 131072 + 64 * 5 + 7)),
    }[name]
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = rng.integers(0, len(deg), int(rp[-1])).astype(np.int32)
    return rp, col


@pytest.mark.parametrize("word4", [False, True])
@pytest.mark.parametrize("tpb", [48, 256, 1024])
@pytest.mark.parametrize("name", ["one", "block_less_one", "block_exact", "block_plus_one",
                                  "round_less_one", "round_exact", "round_plus_one", "empty_rows",
                                  "two_hubs", "wide"])
def test_labelprop_edges(name, tpb, word4):
    import torch
    from paper_2401_04701_amd import hr
    rp, col = graph(name)
    n, m = rp.shape[0] - 1, col.shape[0]
    if word4 and (n + tpb - 1) // tpb > 1 << 14:
        pytest.skip("the graph does not fit the 4-byte word's block field")
    mask = (np.random.default_rng(12).random(m) < 0.03).astype(np.uint8)
    print("[case] labelprop edges", name, "tpb", tpb, "word4", word4, flush=True)
    up = lambda a: torch.from_numpy(a).cuda()
    rp_d, col_d, mask_d = up(rp), up(col), up(mask)
    kw = {"word4": True, "thread_bits": 10} if word4 else {}
    with hr.Context(count_checks=True, ring_capacity=1 << 20, **kw) as ctx:
        label = torch.arange(n, dtype=torch.int32, device="cuda")
        regs = [ctx.shadow_alloc(label), ctx.shadow_alloc(rp_d), ctx.shadow_alloc(col_d)]
        for _ in range(2):
            ctx.labelprop_check(regs[0], label, rp_d, col_d, mask_d, tpb=tpb, r_row_ptr=regs[1],
                                r_col=regs[2])
            ctx.kernel_end()
        got, cnt = ctx.flagged(), ctx.check_count()
        assert ctx.status == 0
    assert cnt == 2 * (3 * n + 2 * m + int(mask.sum()))
    assert got == cf.labelprop_flagged(rp, col, mask)
    if n < 1000:
        log = oracle.model_labelprop(rp, col, mask, 2, tpb, monitor_csr=True)
        assert cnt == log.shape[0] and got == oracle.flagged(log)
    # without races the sweeps converge to the smallest label that reaches a vertex
    src = np.repeat(np.arange(n), np.diff(rp))
    want = np.arange(n, dtype=np.int32)
    while True:
        nxt = want.copy()
        np.minimum.at(nxt, col, want[src])
        if (nxt == want).all():
            break
        want = nxt
    none = torch.zeros_like(mask_d)
    for checked in (False, True):
        label = torch.arange(n, dtype=torch.int32, device="cuda")
        with hr.Context(**kw) as ctx:
            r = ctx.shadow_alloc(label)
            before = None
            while before is None or not torch.equal(before, label):
                before = label.clone()
                if checked:
                    ctx.labelprop_check(r, label, rp_d, col_d, none, tpb=tpb)
                    ctx.kernel_end()
                else:
                    hr.labelprop_plain(label, rp_d, col_d, none, tpb=tpb)
            assert ctx.flagged() == set() and ctx.status == 0
        assert (label.cpu().numpy() == want).all()
