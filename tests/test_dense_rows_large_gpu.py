"""The initial SGM with four path lines per wave above 64 hypotheses at sizes well inside the
rule for it (path steps over the longest line's steps of 2,400 to 8,064, where 2,048 are
asked for), 2 and 4 cross views, wide and tall images: aggregated costs of Eq. (9) of every
cross view, equal to the oracle's (whole numbers).  The last two are too thin for it."""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,W,N,npaths,T,S", [
    (124, 131, 66, 8, 3, 3), (131, 126, 100, 16, 3, 3), (65, 66, 127, 16, 3, 3),
    (128, 128, 128, 8, 3, 3), (75, 303, 70, 8, 3, 3), (303, 75, 70, 8, 3, 3),
    (75, 180, 101, 16, 1, 3), (180, 75, 101, 16, 5, 1), (150, 151, 80, 8, 1, 5),
    (150, 460, 65, 8, 1, 3), (460, 150, 65, 8, 3, 1),
])
def test_dense_rows_large(H, W, N, npaths, T, S):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng = np.random.default_rng(H * W + N)
    views = rng.integers(0, 256, size=(T, S, H, W)).astype(np.uint8)
    hyp = np.linspace(-4.0, 4.5, N).astype(np.float32)
    p = lfsynth._params(census=(7, 9), p_init=(21, 45), p_final=(17, 35), npaths=npaths,
                        sum_bits=32)
    print("dense rows", H, W, N, npaths, T, S, flush=True)
    got = lf.lf_initial_disparity(torch.from_numpy(views).cuda(), torch.from_numpy(hyp).cuda(), p,
                                  want_volumes=True)
    ref = lfo.depth(views, hyp, p, want_intermediates=True, want_initial_volumes=True)
    assert np.array_equal(got["csum_init"].cpu().numpy().view(np.uint16).astype(np.int64),
                          ref["init_csum"])
    assert np.array_equal(got["maps"].cpu().numpy(), ref["maps"])
