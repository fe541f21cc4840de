"""The winner search and the median against the oracle: winners and disparities of given
aggregated costs, bit-exact (the same float32 operations).

Range widths sit around the limits of the search: 8 hypotheses are one round of loads, 32
the widest pixel that a single lane searches, 128 the hypotheses of one round of 16
lanes; costs are small numbers, so that ties are frequent, or the largest ones; maps
are narrower than a workgroup, a window or a median's four rows, and the last pixels'
costs end the volume.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,W,N,widths,sum_bits,top", [
    (37, 61, 100, [7, 7, 7, 100], 32, 40),
    (37, 61, 100, [1, 2, 8, 9, 15, 16, 17, 100], 16, 40),
    (21, 67, 256, [127, 128, 129, 255, 256], 32, 3),
    (21, 67, 40, [31, 32, 33], 16, 20),
    (21, 67, 256, [1, 256], 16, 3),
    (1, 300, 13, [1, 5, 13], 32, 2 ** 32 - 1),
    (301, 1, 17, [16, 17], 16, 2 ** 16 - 1),
    (2, 2, 24, [24], 32, 9),
    (6, 3, 16, [3, 4, 5], 16, 9),
])
def test_wta_ranges(H, W, N, widths, sum_bits, top):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng = np.random.default_rng(H * W + N + sum_bits)
    w = rng.choice(widths, size=(H, W))
    lo = rng.integers(0, N - w + 1).astype(np.int16)
    hi = (lo + w - 1).astype(np.int16)
    off = np.concatenate([[0], np.cumsum(w.reshape(-1))]).astype(np.int64)
    u = np.uint16 if sum_bits == 16 else np.uint32
    csum = rng.integers(max(0, top - 40), top, size=int(off[-1]), endpoint=True).astype(u)
    pix = np.repeat(np.arange(H * W), w.reshape(-1))
    k = lo.reshape(-1)[pix] + (np.arange(off[-1]) - off[:-1][pix])
    dense = np.zeros((H * W, N), dtype=np.int64)
    dense[pix, k] = csum
    dense = dense.reshape(H, W, N)
    hyp = np.linspace(-2.0, 3.0, N).astype(np.float32)
    print("wta ranges", H, W, N, widths, sum_bits, top, flush=True)
    dev = "cuda"
    signed = np.int16 if sum_bits == 16 else np.int32
    got = lf.lf_wta_subpixel(torch.from_numpy(csum.view(signed)).to(dev), sum_bits,
                             torch.from_numpy(off).to(dev), torch.from_numpy(lo).to(dev),
                             torch.from_numpy(hi).to(dev), torch.from_numpy(hyp).to(dev), 3)
    idx = lfo.wta(dense, lo, hi)
    assert np.array_equal(got["d_index"].cpu().numpy(), idx)
    want = lfo.median3(lfo.subpixel(dense, idx, hyp, lo, hi))
    assert np.array_equal(got["disparity"].cpu().numpy(), want)


@pytest.mark.parametrize("H,W", [(9, 70), (3, 3), (5, 1)])
def test_median_with_nan(H, W):
    # a hypothesis that is no number reaches the map; windows without one are unchanged
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng = np.random.default_rng(H + W)
    idx = rng.integers(0, 12, size=(H, W)).astype(np.int16)
    hyp = np.array([-2, -1.5, -0.0, 0.0, np.nan, 0.5, 1, 1.5, 2, np.inf, -np.inf, 3], np.float32)
    n = H * W
    off = np.arange(n + 1, dtype=np.int64)           # one hypothesis per pixel
    dev = "cuda"
    print("median with nan", H, W, flush=True)
    got = lf.lf_wta_subpixel(torch.zeros(n, dtype=torch.int32, device=dev), 32,
                             torch.from_numpy(off).to(dev), torch.from_numpy(idx).to(dev),
                             torch.from_numpy(idx).to(dev), torch.from_numpy(hyp).to(dev), 3)
    x = np.pad(hyp[idx], 1, mode="edge")
    win = np.stack([x[i:i + H, j:j + W] for i in range(3) for j in range(3)])
    below = (win[None] < win[:, None]).sum(1)
    atmost = (win[None] <= win[:, None]).sum(1)
    want = win[4].copy()
    for i in range(9):
        want = np.where((below[i] <= 4) & (atmost[i] > 4), win[i], want)
    assert np.array_equal(got["disparity"].cpu().numpy(), want, equal_nan=True)
