"""Buffers that start at an address of 2 mod 4: 16-bit costs, sums and bounds that are a part
of larger allocations.  Against the oracle, whole numbers, equal.

The bounded SGM with four lines per wave loads words of costs from the 4-byte boundary
before the first one; the winner search loads 8 sums at a time.  The workspace says which
bounded SGM kernel ran."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _part(x):
    """x on the GPU, two bytes into an allocation."""
    buf = torch.zeros(x.size + 3, dtype=torch.int16, device="cuda")
    part = buf[1:1 + x.size].view(x.shape)
    part.copy_(torch.from_numpy(x.view(np.int16)))
    assert part.data_ptr() % 4 == 2
    return part


def _ranges(H, W, N, widths, seed):
    rng = np.random.default_rng(seed)
    w = rng.choice(widths, size=(H, W))
    mid = np.cumsum(rng.integers(-1, 2, size=(H, W)), axis=1) + N // 2
    lo = np.clip(mid, 0, N - w).astype(np.int16)
    hi = (lo + w - 1).astype(np.int16)
    off = np.concatenate([[0], np.cumsum(w.reshape(-1))]).astype(np.int64)
    pix = np.repeat(np.arange(H * W), w.reshape(-1))
    k = lo.reshape(-1)[pix] + (np.arange(off[-1]) - off[:-1][pix])
    return rng, lo, hi, off, pix, k


@pytest.mark.parametrize("H,W,N,npaths,sum_bits,widths,four", [
    (290, 301, 61, 16, 16, [7] * 20 + [15, 61], 1),
    (290, 301, 61, 16, 16, [21], 0),
    (301, 290, 127, 16, 32, [1, 7, 7, 7, 7, 7, 7, 7, 7, 127], 1),
    (301, 300, 255, 8, 16, [5] * 20 + [17, 255], 1),
    (40, 51, 99, 8, 16, [3, 99], 0),
])
def test_bounded_sgm_at_2_mod_4(H, W, N, npaths, sum_bits, widths, four):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng, lo, hi, off, pix, k = _ranges(H, W, N, widths, N)
    P1, P2 = 17, 35
    cap = lfo.cost_cap(P2, npaths, sum_bits)
    cost = rng.integers(0, cap + 1, size=int(off[-1])).astype(np.uint16)
    print("bounded SGM at 2 mod 4", H, W, N, npaths, sum_bits, flush=True)
    ws = lf.workspace(lf.lib.lf_sgm_workspace_size(H, W, N, npaths), "cuda")
    csum = _part(np.zeros(cost.size, np.uint16)) if sum_bits == 16 else None
    csum = lf.lf_sgm_aggregate(_part(cost), torch.from_numpy(off).cuda(), _part(lo), _part(hi),
                               N, P1, P2, npaths, sum_bits, csum=csum, ws=ws)
    got = csum.cpu().numpy().view(np.uint16 if sum_bits == 16 else np.uint32)
    assert int(ws[12:16].view(torch.int32)) == four
    dense = np.zeros((H * W, N), dtype=np.int32)
    dense[pix, k] = cost
    ref = lfo.sgm(dense.reshape(H, W, N), P1, P2, npaths, lo=lo, hi=hi).reshape(H * W, N)
    assert np.array_equal(got.astype(np.int64), ref[pix, k].astype(np.int64))


@pytest.mark.parametrize("H,W,N,widths", [(37, 61, 100, [1, 7, 8, 9, 100]), (9, 70, 32, [31, 32]),
                                          (5, 3, 256, [33, 256])])
def test_winner_search_at_2_mod_4(H, W, N, widths):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng, lo, hi, off, pix, k = _ranges(H, W, N, widths, N)
    csum = rng.integers(0, 300, size=int(off[-1])).astype(np.uint16)
    hyp = np.linspace(-2.0, 3.0, N).astype(np.float32)
    print("winner search at 2 mod 4", H, W, N, flush=True)
    got = lf.lf_wta_subpixel(_part(csum), 16, torch.from_numpy(off).cuda(), _part(lo), _part(hi),
                             torch.from_numpy(hyp).cuda(), 3)
    dense = np.zeros((H * W, N), dtype=np.int64)
    dense[pix, k] = csum
    dense = dense.reshape(H, W, N)
    idx = lfo.wta(dense, lo, hi)
    assert np.array_equal(got["d_index"].cpu().numpy(), idx)
    assert np.array_equal(got["disparity"].cpu().numpy(),
                          lfo.median3(lfo.subpixel(dense, idx, hyp, lo, hi)))
