"""The bounded l2 cost of a volume of 2^34 cells, more than one launch has work items for at
four cells each: every pixel at its full range.  The costs of a sample of pixels (the
first and the last among them) at whole-pixel shifts, where a bilinear sum is the sample
itself: sums of whole numbers, equal."""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_l2_2_34_cells():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_13449_amd import lf
    H, W, N = 8193, 8193, 256
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("needs 64 GB")
    dev = "cuda"
    gen = torch.Generator(dev).manual_seed(9)
    views = torch.randint(0, 256, (1, 3, H, W), dtype=torch.uint8, device=dev, generator=gen)
    hyp = torch.arange(-100, N - 100, dtype=torch.float32, device=dev)
    p = lfsynth._params(alpha=1.0, sum_bits=32)
    lo = torch.zeros((H, W), dtype=torch.int16, device=dev)
    hi = torch.full((H, W), N - 1, dtype=torch.int16, device=dev)
    print("l2 of", H * W * N, "cells", flush=True)
    got = lf.lf_cost_volume_bounded(views, hyp, p, lo, hi)
    assert int(got["offsets"][-1]) == H * W * N
    pix = torch.randint(0, H * W, (20000,), device=dev, generator=gen)
    pix[:2] = torch.tensor([0, H * W - 1])
    cost = got["cost"].view(H * W, N)[pix].cpu().numpy().view(np.uint16)
    img = views[0].cpu().numpy().astype(np.int64)
    pix, d = pix.cpu().numpy(), hyp.cpu().numpy().astype(np.int64)
    v, u = pix[:, None] // W, pix[:, None] % W
    want = sum(np.abs(img[1][v, u] - img[s][v, np.clip(u + (1 - s) * d, 0, W - 1)])
               for s in (0, 2))
    assert np.array_equal(cost, want)
