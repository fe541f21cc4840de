"""The l2 cost of a search without bounds (lambda < 0), whose volume is dense: the whole
method against the oracle, and against the general kernels on the same full ranges.

Sizes: no multiples of the 3 columns, the 2 to 4 rows and the 8 hypotheses that a
workgroup's lanes and waves hold, down to a single column or row.  Values: 8-bit and
float, gray and colour; shifts below 2^-24 and colours scaled so that squares leave the
range of the fast root; pixels that are infinite or no number (against the general
kernels only: their costs are the same expression)."""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,W,N,T,S,C,dtype,scale,odd", [
    (19, 47, 37, 3, 5, 1, "u8", 1, False),
    (19, 47, 37, 3, 5, 1, "f32", 1.0, False),
    (18, 50, 40, 3, 3, 3, "u8", 1, False),
    (17, 49, 15, 3, 3, 3, "f32", 1.0, False),
    (40, 1, 8, 3, 3, 1, "u8", 1, False),
    (1, 200, 256, 1, 3, 1, "f32", 1.0, False),
    (5, 2, 9, 3, 1, 3, "u8", 1, False),
    (13, 21, 12, 3, 3, 3, "f32", 1e-20, False),
    (13, 21, 12, 3, 3, 3, "f32", 1e25, False),
    (19, 47, 20, 3, 5, 1, "f32", 1.0, True),
    (19, 47, 20, 3, 3, 3, "f32", 1.0, True),
])
def test_cost_full_range(H, W, N, T, S, C, dtype, scale, odd):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng = np.random.default_rng(H * W + N + C)
    shape = (T, S, C, H, W) if C == 3 else (T, S, H, W)
    if dtype == "u8":
        views = rng.integers(0, 256, size=shape).astype(np.uint8)
    else:
        views = (rng.random(shape) * scale).astype(np.float32)
    if odd:
        at = rng.random(shape) < 0.02
        views[at] = rng.choice([np.inf, -np.inf, np.nan], size=int(at.sum()))
    hyp = np.linspace(-3.1, 3.3, N).astype(np.float32)
    hyp[N // 2 - 2: N // 2 + 2] = [-2.0 ** -25, 0.0, 2.0 ** -40, 2.0 ** -24]
    p = lfsynth._params(lam=-1, alpha=1.0 if dtype == "u8" else 255.0, sum_bits=32)
    print("cost full range", H, W, N, T, S, C, dtype, scale, odd, flush=True)
    dev = "cuda"
    v, h = torch.from_numpy(views).to(dev), torch.from_numpy(hyp).to(dev)
    got = lf.lf_depth(v, h, p).cpu().numpy()
    lo = torch.zeros((H, W), dtype=torch.int16, device=dev)
    hi = torch.full((H, W), N - 1, dtype=torch.int16, device=dev)
    cv = lf.lf_cost_volume_bounded(v, h, p, lo, hi)
    csum = lf.lf_sgm_aggregate(cv["cost"], cv["offsets"], lo, hi, N, p["P1_final"],
                               p["P2_final"], p["npaths"], p["sum_bits"])
    want = lf.lf_wta_subpixel(csum, p["sum_bits"], cv["offsets"], lo, hi, h, p["median"])
    assert np.array_equal(got, want["disparity"].cpu().numpy())
    if not odd:
        ref = lfo.depth(views, hyp, p)
        assert np.array_equal(got, ref["disparity"])
