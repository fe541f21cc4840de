"""The Census cost volume of the initial stage against the oracle's Eq. (7), whole numbers:
views whose shifts span fewer pixels than there are hypotheses and more, around the limits
of the two ways it is computed (0.65 pixels per hypothesis, 0.8 in colour), both shift
axes, and hypothesis counts that end inside a word of four."""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("C", [1, 3])
@pytest.mark.parametrize("per", [0.1, 0.6, 0.64, 0.67, 0.78, 0.82, 1.3, 4.0])
@pytest.mark.parametrize("H,W,N,S,T", [(21, 67, 41, 5, 3), (40, 33, 100, 3, 5), (9, 130, 6, 3, 1)])
def test_census_volume(H, W, N, S, T, per, C):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng = np.random.default_rng(N + C)
    shape = (T, S, C, H, W) if C == 3 else (T, S, H, W)
    views = rng.integers(0, 256, size=shape).astype(np.uint8)
    reach = per * N / (S // 2) / 2
    hyp = np.linspace(-reach, reach, N).astype(np.float32)
    p = lfsynth._params(census=(5, 5), p_init=(10, 60), p_final=(17, 35), sum_bits=32)
    print("census volume", H, W, N, S, T, per, C, flush=True)
    got = lf.lf_initial_disparity(torch.from_numpy(views).cuda(), torch.from_numpy(hyp).cuda(), p,
                                  want_volumes=True)
    ref = lfo.depth(views, hyp, p, want_intermediates=True, want_initial_volumes=True)
    assert np.array_equal(got["census_cost"].cpu().numpy().astype(np.int32), ref["init_cost"])
