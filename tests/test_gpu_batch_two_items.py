"""Batched label propagation in jobs of exactly two work items a phase, many
phases, beside jobs of other sizes: labels and flagged sets."""
import numpy as np
import pytest

from oracle import closed_forms as cf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [0, 1])
def test_two_items_a_phase(variant):
    import torch
    from paper_2401_04701_amd import hr
    print("[case] two items a phase, variant", variant, flush=True)
    rng = np.random.default_rng(4)
    jobs, want = [], []
    for j in range(60):
        n = [1100, 1999, 2048, 500, 3000][j % 5]          # 2, 2, 2, 1, 3 items of 1,024
        deg = rng.integers(0, 6, n)
        deg[rng.integers(0, n)] = 700
        rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
        col = rng.integers(0, n, int(rp[-1])).astype(np.int32)
        mask = (rng.random(col.shape[0]) < 0.01 * (j % 2)).astype(np.uint8)
        t = [torch.arange(n, dtype=torch.int32, device="cuda")]
        t += [torch.from_numpy(a).cuda() for a in (rp, col, mask)]
        inst = hr.Instance()
        inst.drop = -1
        inst.region[0] = inst.region[1] = hr.NO_REGION
        inst.pattern, inst.phases, inst.n, inst.threads = hr.HR_PAT_LABELPROP, 40, n, 64
        for i, x in enumerate(t):
            inst.data[i] = x.data_ptr()
        jobs.append((inst, t))
        fixed = np.arange(n, dtype=np.int32)
        src = np.repeat(np.arange(n), np.diff(rp))
        while True:
            nxt = fixed.copy()
            np.minimum.at(nxt, col, fixed[src])
            if (nxt == fixed).all():
                break
            fixed = nxt
        want.append((fixed if not mask.any() else None, cf.labelprop_flagged(rp, col, mask)))
    with hr.Context(ring_capacity=1 << 18) as ctx:
        with hr.Batch(ctx, [j[0] for j in jobs]) as b:
            b.run(variant=variant)
            got = b.split(ctx.flagged())
            assert ctx.status == 0
    for (inst, t), (fixed, flagged), g in zip(jobs, want, got):
        assert set(g) == flagged
        if fixed is not None:
            assert (t[0].cpu().numpy() == fixed).all()
