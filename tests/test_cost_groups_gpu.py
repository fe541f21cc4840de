"""The bounded l2 cost of groups of adjacent pixels, against the oracle's sums of
Eq. (12): the float32 sums bit-exact (same operations in the same order).

Sizes: rows that are no multiple of a group (3 pixels), shorter than one or a single
pixel, windows that jump between neighbours (a group's hull has gaps), slices that end
inside a group (2 and, above 2^26 cells at most, 4 cells per thread).  Values: shifts
below 2^-24, where 8-bit colour sums take the exact square root, and colour views scaled
so that squares leave the range of the fast root (underflow, overflow).
"""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,W,N,T,S,C,dtype,scale,widths", [
    (33, 61, 40, 3, 5, 1, "u8", 1, [7, 7, 40]),
    (33, 61, 40, 3, 5, 3, "u8", 1, [1, 7, 40]),
    (31, 62, 40, 3, 3, 3, "f32", 1.0, [7, 7, 40]),
    (40, 1, 256, 3, 3, 1, "f32", 1.0, [1, 2, 256]),
    (40, 2, 100, 1, 3, 3, "u8", 1, [1, 100]),
    (1, 300, 13, 3, 1, 1, "u8", 1, [1, 3, 13]),
    (21, 43, 30, 3, 3, 3, "f32", 1e-20, [5, 30]),       # squares underflow
    (21, 43, 30, 3, 3, 3, "f32", 1e25, [5, 30]),        # squares overflow
    (530, 523, 256, 1, 3, 1, "u8", 1, [1, 3]),          # 4 cells per thread
    (530, 523, 256, 1, 3, 3, "u8", 1, [1, 3]),
])
def test_cost_groups(H, W, N, T, S, C, dtype, scale, widths):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng = np.random.default_rng(H * W + N + C)
    shape = (T, S, C, H, W) if C == 3 else (T, S, H, W)
    if dtype == "u8":
        views = rng.integers(0, 256, size=shape).astype(np.uint8)
        views[..., : W // 2] = views[:1, :1, ..., : W // 2]     # sums that are 0
    else:
        views = (rng.random(shape) * scale).astype(np.float32)
        views[..., : H // 2, :] = views[:1, :1, ..., : H // 2, :]
    hyp = np.linspace(-3.1, 3.3, N).astype(np.float32)
    hyp[N // 2 - 3: N // 2 + 3] = [-2.0 ** -23, -2.0 ** -25, 0.0, 2.0 ** -40, 2.0 ** -24, 1.0]
    w = rng.choice(widths, size=(H, W))
    mid = np.cumsum(rng.integers(-1, 2, size=(H, W)), axis=1) + N // 2
    mid = np.where(rng.random((H, W)) < 0.1, rng.integers(0, N, size=(H, W)), mid)
    lo = np.clip(mid, 0, N - w).astype(np.int16)
    hi = (lo + w - 1).astype(np.int16)
    p = lfsynth._params(alpha=255.0 if dtype == "f32" else 1.0, sum_bits=16)
    print("cost groups", H, W, N, T, S, C, dtype, scale, flush=True)
    dev = "cuda"
    got = lf.lf_cost_volume_bounded(
        torch.from_numpy(views).to(dev), torch.from_numpy(hyp).to(dev), p,
        torch.from_numpy(lo).to(dev), torch.from_numpy(hi).to(dev), want_f32=True)
    off = got["offsets"].cpu().numpy()
    n = hi.astype(np.int64).reshape(-1) - lo.reshape(-1) + 1
    assert np.array_equal(off, np.concatenate([[0], np.cumsum(n)]))
    pix = np.repeat(np.arange(H * W), n)
    k = lo.reshape(-1)[pix] + (np.arange(off[-1]) - off[:-1][pix])
    ref = lfo.cost_l2_f32(views, hyp, lo, hi)
    want = ref.reshape(H * W, N)[pix, k]
    assert np.array_equal(got["cost_f32"].cpu().numpy()[: off[-1]], want)
    cap = lfo.cost_cap(p["P2_final"], p["npaths"], p["sum_bits"])
    quant = lfo.quantize(ref, p["alpha"], cap, lo, hi).reshape(H * W, N)[pix, k]
    assert np.array_equal(got["cost"].cpu().numpy().view(np.uint16)[: off[-1]].astype(np.int64),
                          quant.astype(np.int64))
