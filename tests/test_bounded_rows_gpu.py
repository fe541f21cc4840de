"""The bounded SGM with four path lines per wave, against the oracle's aggregated cost of
Eq. (8)-(9) on identical random costs: bit-exact (integer arithmetic).

The sizes give enough lines for that schedule to be taken (path steps over the longest
line's steps above 4,500, or 2,300 beyond 128 hypotheses; smaller images take it in the
batches of test_batch_gpu.py with bounded_lanes = 16), and the window widths sit around
its limits: 14 hypotheses is the widest narrow window, 15 to 17 the narrowest wide ones;
64, 128 and 256 the ends of the three register layouts, odd numbers of cells in every
one.  Windows also jump further than the 16 lanes of a line between neighbouring pixels.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,W,N,npaths,sum_bits,P1,P2,widths", [
    (290, 301, 100, 16, 32, 17, 35, [7, 7, 7, 100]),
    (301, 283, 70, 16, 16, 17, 35, [1, 7, 13, 14, 15, 16, 17, 70]),   # taller than wide
    (285, 403, 64, 16, 32, 6, 48, [3, 14, 64]),
    (570, 565, 12, 8, 16, 6, 48, [1, 5, 12]),                           # never wide
    (291, 289, 255, 8, 32, 17, 35, [7, 40, 250, 255]),
    (289, 300, 256, 8, 32, 9, 16000, [9, 13, 256]),                     # largest path costs
    (283, 300, 128, 16, 32, 17, 35, [128]),                             # only full ranges
])
def test_bounded_rows(H, W, N, npaths, sum_bits, P1, P2, widths):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng = np.random.default_rng(H * W + N)
    w = rng.choice(widths, size=(H, W))
    # windows that wander slowly, with jumps
    mid = np.cumsum(rng.integers(-1, 2, size=(H, W)), axis=1) + N // 2
    mid = np.where(rng.random((H, W)) < 0.05, rng.integers(0, N, size=(H, W)), mid)
    lo = np.clip(mid, 0, N - w).astype(np.int16)
    hi = (lo + w - 1).astype(np.int16)
    widths64 = hi.astype(np.int64) - lo + 1
    off = np.concatenate([[0], np.cumsum(widths64.reshape(-1))]).astype(np.int64)
    cap = lfo.cost_cap(P2, npaths, sum_bits)
    pix = np.repeat(np.arange(H * W), widths64.reshape(-1))
    k = lo.reshape(-1)[pix] + (np.arange(off[-1]) - off[:-1][pix])
    cost = rng.integers(0, cap + 1, size=int(off[-1])).astype(np.uint16)
    print("bounded rows", H, W, N, npaths, sum_bits, P1, P2, flush=True)
    dev = "cuda"
    csum = lf.lf_sgm_aggregate(torch.from_numpy(cost.view(np.int16)).to(dev),
                               torch.from_numpy(off).to(dev), torch.from_numpy(lo).to(dev),
                               torch.from_numpy(hi).to(dev), N, P1, P2, npaths, sum_bits)
    got = csum.cpu().numpy().view(np.uint16 if sum_bits == 16 else np.uint32)
    dense = np.zeros((H * W, N), dtype=np.int32)
    dense[pix, k] = cost
    ref = lfo.sgm(dense.reshape(H, W, N), P1, P2, npaths, lo=lo, hi=hi).reshape(H * W, N)
    assert np.array_equal(got.astype(np.int64), ref[pix, k].astype(np.int64))
