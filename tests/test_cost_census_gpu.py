"""The bounded Census cost in slices of 512 cells against the oracle's Eq. (15): whole
numbers, equal.  Slices of one pixel and less (256 hypotheses), of many narrow pixels,
images narrower than a slice's pixels, a last slice that is not full."""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,W,N,T,S,C,widths", [
    (23, 41, 64, 3, 5, 1, [1, 7, 64]),
    (40, 37, 256, 1, 3, 1, [256]),
    (17, 31, 100, 3, 1, 3, [1, 100]),
    (700, 1, 20, 1, 3, 1, [1]),
    (1, 3, 9, 3, 3, 3, [9]),
])
def test_cost_census(H, W, N, T, S, C, widths):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng = np.random.default_rng(H * W + N + C)
    views = rng.integers(0, 256, size=(T, S, C, H, W)).astype(np.uint8)
    hyp = np.linspace(-3.1, 3.3, N).astype(np.float32)
    w = rng.choice(widths, size=(H, W))
    lo = rng.integers(0, N - w + 1).astype(np.int16)
    hi = (lo + w - 1).astype(np.int16)
    p = lfsynth._params(cost_kind=1, sum_bits=32)
    cap = lfo.cost_cap(p["P2_final"], p["npaths"], p["sum_bits"])
    print("cost census", H, W, N, T, S, C, flush=True)
    dev = "cuda"
    got = lf.lf_cost_volume_bounded(
        torch.from_numpy(views if C == 3 else views[:, :, 0]).to(dev),
        torch.from_numpy(hyp).to(dev), p, torch.from_numpy(lo).to(dev),
        torch.from_numpy(hi).to(dev), want_f32=True)
    census = np.stack([lfo.census(x.astype(np.float32), p["win_h"], p["win_w"])
                       for x in views.reshape(-1, H, W)]).reshape(T, S, C, H, W)
    ref = lfo.cost_census_all(census if C == 3 else census[:, :, 0], hyp, cap, lo, hi)
    off = got["offsets"].cpu().numpy()
    pix = np.repeat(np.arange(H * W), w.reshape(-1))
    k = lo.reshape(-1)[pix] + (np.arange(off[-1]) - off[:-1][pix])
    want = ref.reshape(H * W, N)[pix, k]
    assert np.array_equal(got["cost"].cpu().numpy().view(np.uint16)[: off[-1]], want)
    assert np.array_equal(np.minimum(got["cost_f32"].cpu().numpy()[: off[-1]], cap), want)
