"""The bounded costs where pixels own no cells (d_hi = d_lo - 1), against the oracle: a
pixel's costs are its own however many empty ranges lie between it and the one before.
The sums of Eq. (12) bit-exact, the costs of Eq. (15) whole numbers, equal.

A slice of the volume holds 512 cells and 512 pixels of it are staged: runs of fewer,
exactly as many and several times as many empty ranges, at the start, inside a slice and
at the end; every range empty."""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _run(kind, C, dtype, H, W, N, keep, seed):
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng = np.random.default_rng(seed)
    T, S = 3, 3
    views = rng.integers(0, 256, size=(T, S, C, H, W)).astype(np.uint8)
    if dtype == "f32":
        views = (views / 255.0).astype(np.float32)
    views = views if C == 3 else views[:, :, 0]
    hyp = np.linspace(-3.1, 3.3, N).astype(np.float32)
    w = rng.choice([1, 5, N], size=H * W)
    w = np.where(keep, w, 0).reshape(H, W)
    lo = rng.integers(0, N - np.maximum(w, 1) + 1).astype(np.int16)
    hi = (lo + w - 1).astype(np.int16)
    p = lfsynth._params(cost_kind=1 if kind == "census" else 0, sum_bits=32,
                        alpha=255.0 if dtype == "f32" else 1.0)
    cap = lfo.cost_cap(p["P2_final"], p["npaths"], p["sum_bits"])
    print("empty ranges", kind, C, dtype, H, W, N, int((w == 0).sum()), flush=True)
    dev = "cuda"
    got = lf.lf_cost_volume_bounded(
        torch.from_numpy(np.ascontiguousarray(views)).to(dev), torch.from_numpy(hyp).to(dev), p,
        torch.from_numpy(lo).to(dev), torch.from_numpy(hi).to(dev), want_f32=True)
    off = got["offsets"].cpu().numpy()
    assert np.array_equal(off, np.concatenate([[0], np.cumsum(w.reshape(-1))]))
    pix = np.repeat(np.arange(H * W), w.reshape(-1))
    k = lo.reshape(-1)[pix] + (np.arange(off[-1]) - off[:-1][pix])
    full = np.zeros((H, W), np.int16), np.full((H, W), N - 1, np.int16)
    cost = got["cost"].cpu().numpy().view(np.uint16)[: off[-1]].astype(np.int64)
    raw = got["cost_f32"].cpu().numpy()[: off[-1]]
    if kind == "census":
        census = np.stack([lfo.census(x.astype(np.float32), p["win_h"], p["win_w"])
                           for x in views.reshape(-1, H, W)]).reshape(views.shape)
        want = lfo.cost_census_all(census, hyp, cap, *full).reshape(H * W, N)[pix, k]
        assert np.array_equal(cost, want)
        assert np.array_equal(np.minimum(raw, cap), want)
    else:
        ref = lfo.cost_l2_f32(views, hyp, *full)
        assert np.array_equal(raw, ref.reshape(H * W, N)[pix, k])
        quant = lfo.quantize(ref, p["alpha"], cap, *full).reshape(H * W, N)[pix, k]
        assert np.array_equal(cost, quant.astype(np.int64))


def _keep(H, W, runs):
    keep = np.ones(H * W, dtype=bool)
    for a, n in runs:
        keep[a:a + n] = False
    return keep


RUNS = {
    "inside": [(40, 511), (700, 512), (1300, 513), (1900, 2600)],
    "ends": [(0, 1700), (4000, 4000)],
    "one": [(0, 2000), (2001, 9999)],
    "none": [(0, 9999)],
}


@pytest.mark.parametrize("runs", list(RUNS))
@pytest.mark.parametrize("C", [1, 3])
def test_empty_ranges_census(C, runs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    H, W, N = 71, 67, 12
    _run("census", C, "u8", H, W, N, _keep(H, W, RUNS[runs]), 5)


@pytest.mark.parametrize("runs", list(RUNS))
@pytest.mark.parametrize("C,dtype", [(1, "u8"), (1, "f32"), (3, "u8"), (3, "f32")])
def test_empty_ranges_l2(C, dtype, runs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    H, W, N = 71, 67, 12
    _run("l2", C, dtype, H, W, N, _keep(H, W, RUNS[runs]), 6)
