"""Batches with several members of the kernels that one light field of the other batch tests
takes at most: searches without bounds (gray and colour, 8-bit and float) and the l2 cost
of 8-bit colour views.  Each result equals that of the light field alone and the oracle's."""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (H, W, N, channels, dtype, parameters)
SETS = {
    "no bounds, gray": [(30, 41, 20, 1, "f32", dict(lam=-1)), (52, 33, 9, 1, "f32", dict(lam=-1)),
                        (37, 40, 64, 1, "u8", dict(lam=-1)), (9, 61, 33, 1, "u8", dict(lam=-1))],
    "no bounds, colour": [(30, 41, 20, 3, "f32", dict(lam=-1)), (22, 33, 9, 3, "f32", dict(lam=-1)),
                          (37, 40, 40, 3, "u8", dict(lam=-1)), (9, 61, 17, 3, "u8", dict(lam=-1))],
    "8-bit colour": [(44, 50, 30, 3, "u8", dict(lam=2)), (31, 70, 60, 3, "u8", dict(lam=4)),
                     (20, 21, 130, 3, "u8", dict(lam=1, npaths=16))],
    "both": [(44, 50, 30, 3, "u8", dict(lam=2)), (30, 41, 20, 3, "u8", dict(lam=-1)),
             (52, 33, 40, 1, "f32", dict(lam=-1)), (40, 40, 24, 1, "f32", dict(lam=3)),
             (33, 30, 24, 3, "f32", dict(lam=3))],
}


@pytest.mark.parametrize("tuning", [None, dict(cost_cells_per_thread=4, cost_stride=2,
                                               bounded_lanes=16)])
@pytest.mark.parametrize("name", list(SETS))
def test_members(name, tuning):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    items, alone, refs = [], [], []
    for i, (H, W, N, C, dtype, p) in enumerate(SETS[name]):
        lfd = lfsynth.workload("paper_s", seed=90 + i, H=H, W=W, S=3, T=5, N=N, channels=C)
        views, prm = lfd.views, dict(lfd.params, sum_bits=32, win_h=5, win_w=5, **p)
        if dtype == "u8":
            views = np.clip(np.rint(views * 255.0), 0, 255).astype(np.uint8)
            prm.update(alpha=1.0, edge_tau=60.0)
        refs.append(lfo.depth(views, lfd.hyp, prm))
        v, h = torch.from_numpy(np.ascontiguousarray(views)).cuda(), torch.from_numpy(lfd.hyp).cuda()
        idx = torch.empty((H, W), dtype=torch.int16, device="cuda")
        alone.append((lf.lf_depth(v, h, prm, d_index=idx), idx))
        items.append((v, h, prm, torch.empty((H, W), device="cuda"),
                      torch.empty((H, W), dtype=torch.int16, device="cuda")))
    plan = lf.Plan(items, tuning=tuning)
    plan.capture()
    for rep in range(3):
        for it in items:
            it[3].fill_(float("nan"))
            it[4].fill_(-7)
        torch.cuda.synchronize()
        print("members", name, tuning, "replay", rep, flush=True)
        plan.run()
        torch.cuda.synchronize()
        for it, (disp, idx), ref in zip(items, alone, refs):
            assert torch.equal(it[3], disp)
            assert torch.equal(it[4], idx)
            assert np.array_equal(it[4].cpu().numpy(), ref["d_index"])
            assert np.array_equal(it[3].cpu().numpy(), ref["disparity"])
