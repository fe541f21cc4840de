"""A batch whose light fields differ in everything that selects a kernel: view type and
channels, Census window, cost kind, fill passes, bounds, hypotheses per lane, 8- and 16-bit
path costs, 8 and 16 paths, both sum widths, with and without the median.  Its plan has a
launch per kernel variant; however many those are, the batch is accepted, and every result
equals that of the light field alone.

Without a GPU a plan ends at the upload of its tables, after it has laid them out."""
import ctypes

import numpy as np
import pytest

import lfsynth

torch = pytest.importorskip("torch")

H, W, S = 18, 21, 3


def _variants():
    """(dtype, channels, N, parameters) of each light field."""
    base = dict(win_h=5, win_w=5, P1_init=10, P2_init=60, P1_final=5, P2_final=20, npaths=8,
                phi=3, lam=2, fill_passes=2, edge_tau=1e9, alpha=1.0, cost_kind=0, median=3,
                sum_bits=32)
    out = []
    for dtype in ("u8", "f32"):
        for C in (1, 3):
            def add(N=10, **p):
                out.append((dtype, C, N, dict(base, **p)))
            sparse = lfsynth.checkerboard_census_offsets(5, 5)
            for window in (dict(), dict(win_h=7, win_w=9), dict(win_h=3, win_w=3),
                           dict(census_offsets=sparse)):
                for kind in (0, 1):
                    add(cost_kind=kind, **window)
            for passes in range(9):
                add(fill_passes=passes)
            add(lam=-1)
            add(lam=-1, cost_kind=1)
    for N in (10, 64, 65, 128, 129, 192, 193, 256):
        for P1, P2 in ((10, 60), (60, 250), (10, 200)):
            for npaths, sum_bits, median in ((8, 16, 0), (8, 32, 3), (16, 16, 3), (16, 32, 0)):
                out.append(("u8", 1, N, dict(base, P1_init=P1, P2_init=P2, npaths=npaths,
                                             sum_bits=sum_bits, median=median)))
    return out


def test_tables_have_room():
    if torch.cuda.is_available():
        pytest.skip("covered by the batch itself")
    from paper_1907_13449_amd import lf
    reqs = []
    for dtype, C, N, p in _variants():
        r = lf.Request()
        r.views = lf.ViewSet(1 << 20, S, S, H, W, W, lf.LF_U8 if dtype == "u8" else lf.LF_F32, C)
        r.hyp, r.N, r.params = 1 << 20, N, lf.make_params(p)
        r.disparity = 1 << 20
        reqs.append(r)
    for order in (reqs, reqs[::7], reqs[:1], reqs[:3]):
        arr = (lf.Request * len(order))(*order)
        need = lf.lib.lf_batch_workspace_size(arr, len(order))
        assert need > 0
        plan = ctypes.c_void_p()
        st = lf.lib.lf_plan_create(arr, len(order), ctypes.c_void_p(1 << 30),
                                   ctypes.c_size_t(need), None, None, ctypes.byref(plan))
        # no device: the upload fails, with everything before it done
        assert st == lf.LF_EDEVICE, lf.lib.lf_last_error()


@pytest.mark.gpu
def test_every_variant_in_one_batch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_13449_amd import lf
    rng = np.random.default_rng(3)
    items, alone = [], []
    for dtype, C, N, p in _variants():
        shape = (S, S, C, H, W) if C == 3 else (S, S, H, W)
        views = rng.integers(0, 256, size=shape).astype(np.uint8)
        if dtype == "f32":
            views = (views / 255.0).astype(np.float32)
            p = dict(p, alpha=255.0)
        views = torch.from_numpy(views).cuda()
        hyp = torch.linspace(-1.5, 1.5, N).cuda()
        idx = torch.empty((H, W), dtype=torch.int16, device="cuda")
        alone.append((lf.lf_depth(views, hyp, p, d_index=idx), idx))
        items.append((views, hyp, p, torch.full((H, W), float("nan"), device="cuda"),
                      torch.full((H, W), -7, dtype=torch.int16, device="cuda")))
    plan = lf.Plan(items)
    print("batch of", len(items), "in", plan.launches, "launches", flush=True)
    assert plan.launches > 64
    plan.run()
    torch.cuda.synchronize()
    for (disp, idx), it in zip(alone, items):
        assert torch.equal(idx, it[4]), it[2]
        assert torch.equal(disp, it[3]), it[2]
