"""The bounded l2 cost where neighbouring pixels' windows have little in common, against the
oracle's sums of Eq. (12): the float32 sums bit-exact.

Windows anywhere among the hypotheses (each slice takes its cells one by one), over some of
the image only (slices of both kinds, and slices that are nearly), in slices of 512 cells
and of 1,024 (above 2^26 cells at most); rows of one and two pixels."""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("C,dtype", [(1, "u8"), (1, "f32"), (3, "f32"), (3, "u8")])
@pytest.mark.parametrize("H,W,N,T,S,widths,share", [
    (33, 61, 64, 3, 5, [7], 1.0),
    (45, 53, 100, 3, 3, [1, 7, 100], 0.5),
    (60, 47, 90, 1, 3, [5, 9], 0.2),
    (300, 1, 40, 3, 1, [3, 40], 0.7),
    (150, 2, 256, 1, 3, [2, 30], 0.7),
    (530, 523, 256, 1, 3, [2], 1.0),                 # slices of 1,024 cells
])
def test_scattered_windows(H, W, N, T, S, widths, share, C, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng = np.random.default_rng(H * W + N + C)
    shape = (T, S, C, H, W) if C == 3 else (T, S, H, W)
    views = rng.integers(0, 256, size=shape).astype(np.uint8)
    if dtype == "f32":
        views = rng.random(shape).astype(np.float32)
    hyp = np.linspace(-3.1, 3.3, N).astype(np.float32)
    w = rng.choice(widths, size=(H, W))
    mid = np.where(rng.random((H, W)) < share, rng.integers(0, N, size=(H, W)), N // 2)
    lo = np.clip(mid, 0, N - w).astype(np.int16)
    hi = (lo + w - 1).astype(np.int16)
    p = lfsynth._params(alpha=255.0 if dtype == "f32" else 1.0, sum_bits=32)
    print("scattered windows", H, W, N, T, S, C, dtype, flush=True)
    dev = "cuda"
    got = lf.lf_cost_volume_bounded(
        torch.from_numpy(views).to(dev), torch.from_numpy(hyp).to(dev), p,
        torch.from_numpy(lo).to(dev), torch.from_numpy(hi).to(dev), want_f32=True)
    off = got["offsets"].cpu().numpy()
    pix = np.repeat(np.arange(H * W), w.reshape(-1))
    k = lo.reshape(-1)[pix] + (np.arange(off[-1]) - off[:-1][pix])
    ref = lfo.cost_l2_f32(views, hyp, lo, hi)
    assert np.array_equal(got["cost_f32"].cpu().numpy()[: off[-1]],
                          ref.reshape(H * W, N)[pix, k])
    cap = lfo.cost_cap(p["P2_final"], p["npaths"], p["sum_bits"])
    quant = lfo.quantize(ref, p["alpha"], cap, lo, hi).reshape(H * W, N)[pix, k]
    assert np.array_equal(got["cost"].cpu().numpy().view(np.uint16)[: off[-1]].astype(np.int64),
                          quant.astype(np.int64))
