"""The bounded SGM with four path lines per wave where narrow and wide pixels alternate, so
that a pixel's path costs reach the next one through LDS at nearly every step: as words,
as single entries over a fill, and as single entries read back.  Against the oracle's
aggregated cost of Eq. (8)-(9) on identical random costs: bit-exact.

Path steps over the longest line's steps are 11,120, enough for that schedule whatever the
ranges; the workspace says which ran."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,widths,period", [
    (40, [5, 20], 1),             # two registers per lane: narrow, wide, narrow, ...
    (64, [14, 15, 64], 1),        # the narrowest wide window beside the widest narrow one
    (100, [7, 33, 100], 1),       # four registers per lane
    (90, [9, 40, 41], 2),         # two pixels each: from wide windows to others
])
def test_alternating_windows(N, widths, period):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    H, W, npaths, P1, P2 = 700, 695, 16, 17, 700
    rng = np.random.default_rng(N)
    v, u = np.mgrid[0:H, 0:W]
    w = np.array(widths)[(u // period + v // period) % len(widths)]
    mid = np.cumsum(rng.integers(-2, 3, size=(H, W)), axis=1) + N // 2
    mid = np.where(rng.random((H, W)) < 0.05, rng.integers(0, N, size=(H, W)), mid)
    lo = np.clip(mid, 0, N - w).astype(np.int16)
    hi = (lo + w - 1).astype(np.int16)
    off = np.concatenate([[0], np.cumsum(w.reshape(-1))]).astype(np.int64)
    pix = np.repeat(np.arange(H * W), w.reshape(-1))
    k = lo.reshape(-1)[pix] + (np.arange(off[-1]) - off[:-1][pix])
    cost = rng.integers(0, 3000, size=int(off[-1])).astype(np.uint16)
    print("alternating windows", N, widths, period, flush=True)
    dev = "cuda"
    ws = lf.workspace(lf.lib.lf_sgm_workspace_size(H, W, N, npaths), dev)
    csum = lf.lf_sgm_aggregate(torch.from_numpy(cost.view(np.int16)).to(dev),
                               torch.from_numpy(off).to(dev), torch.from_numpy(lo).to(dev),
                               torch.from_numpy(hi).to(dev), N, P1, P2, npaths, 32, ws=ws)
    assert int(ws[12:16].view(torch.int32)) == 1     # four lines per wave
    dense = np.zeros((H * W, N), dtype=np.int32)
    dense[pix, k] = cost
    ref = lfo.sgm(dense.reshape(H, W, N), P1, P2, npaths, lo=lo, hi=hi).reshape(H * W, N)
    got = csum.cpu().numpy().view(np.uint32)[: off[-1]]
    assert np.array_equal(got.astype(np.int64), ref[pix, k].astype(np.int64))
