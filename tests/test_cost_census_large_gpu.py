"""The bounded Census cost of a volume of 2^33 cells, more than one launch has work items for
at a cell each: every pixel at its full range, so that each workgroup walks several slices.
The costs of a sample of pixels (the first and the last among them) against the Hamming
distances of the library's own strings (tested elsewhere), whole numbers."""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_census_2_33_cells():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_13449_amd import lf
    H, W, N = 5793, 5793, 256
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GB")
    dev = "cuda"
    gen = torch.Generator(dev).manual_seed(9)
    views = torch.randint(0, 256, (1, 3, H, W), dtype=torch.uint8, device=dev, generator=gen)
    hyp = torch.linspace(-40.0, 41.0, N, device=dev)
    p = lfsynth._params(cost_kind=1, sum_bits=32)
    lo = torch.zeros((H, W), dtype=torch.int16, device=dev)
    hi = torch.full((H, W), N - 1, dtype=torch.int16, device=dev)
    print("census of", H * W * N, "cells", flush=True)
    got = lf.lf_cost_volume_bounded(views, hyp, p, lo, hi)
    assert int(got["offsets"][-1]) == H * W * N
    pix = torch.randint(0, H * W, (20000,), device=dev, generator=gen)
    pix[:2] = torch.tensor([0, H * W - 1])
    cost = got["cost"].view(H * W, N)[pix].cpu().numpy().view(np.uint16)
    strings = [lf.lf_census(views[0, s], p["win_h"], p["win_w"]).cpu().numpy().view(np.uint64)
               for s in range(3)]
    pix, hyp = pix.cpu().numpy(), hyp.cpu().numpy()
    v, u = pix // W, pix % W
    want = np.zeros((len(pix), N), dtype=np.int64)
    for s in range(3):
        x = np.clip(u[:, None] + np.rint(np.float32(1 - s) * hyp).astype(np.int64), 0, W - 1)
        diff = strings[1][v, u][:, None] ^ strings[s][v[:, None], x]
        want += np.unpackbits(diff.view(np.uint8).reshape(len(pix), N, 8), axis=2).sum(2, dtype=np.int64)
    cap = lf.cost_cap(p["P2_final"], p["npaths"], p["sum_bits"])
    assert np.array_equal(cost, np.minimum(want, cap))
