"""The bounded l2 cost of 8-bit gray views at widths around multiples of 128, where the rows
of the view copy are lengthened, against the oracle's sums of Eq. (12): the float32 sums
bit-exact.  Shifts reach past both margins; up to 7 rows and 63 columns are left alone."""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,W", [(9, w) for w in (63, 64, 112, 113, 118, 121, 122, 125, 131, 132,
                                                  240, 241, 250, 259, 260, 506, 512)]
                         + [(7, 122), (8, 122), (3, 250)])
def test_cost_widths(H, W):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    N, T, S = 24, 3, 3
    rng = np.random.default_rng(H * W)
    views = rng.integers(0, 256, size=(T, S, H, W)).astype(np.uint8)
    hyp = np.linspace(-W * 1.1, W * 1.1, N).astype(np.float32)
    hyp[N // 2 - 8: N // 2 + 8] = np.linspace(-4.2, 4.4, 16)
    lo = np.zeros((H, W), np.int16)
    hi = np.full((H, W), N - 1, np.int16)
    p = lfsynth._params(alpha=1.0, sum_bits=32)
    print("cost widths", H, W, flush=True)
    got = lf.lf_cost_volume_bounded(torch.from_numpy(views).cuda(), torch.from_numpy(hyp).cuda(),
                                    p, torch.from_numpy(lo).cuda(), torch.from_numpy(hi).cuda(),
                                    want_f32=True)
    ref = lfo.cost_l2_f32(views, hyp, lo, hi)
    assert np.array_equal(got["cost_f32"].cpu().numpy().reshape(H, W, N), ref)
    # and without bounds
    disp = lf.lf_depth(torch.from_numpy(views).cuda(), torch.from_numpy(hyp).cuda(),
                       dict(p, lam=-1))
    want = lfo.depth(views, hyp, dict(p, lam=-1))
    assert np.array_equal(disp.cpu().numpy(), want["disparity"])
