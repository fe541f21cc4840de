"""Which bounded SGM kernel runs (a path line per wave, or four), and that both give the
oracle's aggregated cost of Eq. (8)-(9) on identical random costs: bit-exact.

Between the sizes where four lines per wave never pay and those where they always do the
ranges decide, on the GPU: mostly narrow windows (up to 14 hypotheses) take four lines, wide
ones of few cells one, full ranges of many cells four.  The first pixel's entry in the
workspace says which ran.  The sizes from which four lines are taken whatever the ranges are
path steps over the longest line's steps of 11,000 (up to 128 hypotheses), 16,000 (up to
192) and 9,000."""
import numpy as np
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _run(H, W, N, npaths, sum_bits, P1, P2, widths, share=None, jump=0.05):
    """The flag of the workspace; the sums compared.  widths: drawn per pixel, or per block
    of 8 x 8 pixels the second with probability `share`."""
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    rng = np.random.default_rng(H * W + N)
    if share is None:
        w = rng.choice(widths, size=(H, W))
    else:
        block = rng.random((H // 8 + 1, W // 8 + 1)) < share
        block = np.kron(block, np.ones((8, 8), dtype=bool))[:H, :W]
        w = np.where(block, widths[1], widths[0])
    mid = np.cumsum(rng.integers(-1, 2, size=(H, W)), axis=1) + N // 2
    mid = np.where(rng.random((H, W)) < jump, rng.integers(0, N, size=(H, W)), mid)
    lo = np.clip(mid, 0, N - w).astype(np.int16)
    hi = (lo + w - 1).astype(np.int16)
    off = np.concatenate([[0], np.cumsum(w.reshape(-1))]).astype(np.int64)
    cap = lfo.cost_cap(P2, npaths, sum_bits)
    pix = np.repeat(np.arange(H * W), w.reshape(-1))
    k = lo.reshape(-1)[pix] + (np.arange(off[-1]) - off[:-1][pix])
    cost = rng.integers(0, cap + 1, size=int(off[-1])).astype(np.uint16)
    print("bounded choice", H, W, N, npaths, sum_bits, P1, P2, widths, share, flush=True)
    dev = "cuda"
    ws = lf.workspace(lf.lib.lf_sgm_workspace_size(H, W, N, npaths), dev)
    csum = lf.lf_sgm_aggregate(torch.from_numpy(cost.view(np.int16)).to(dev),
                               torch.from_numpy(off).to(dev), torch.from_numpy(lo).to(dev),
                               torch.from_numpy(hi).to(dev), N, P1, P2, npaths, sum_bits, ws=ws)
    got = csum.cpu().numpy().view(np.uint16 if sum_bits == 16 else np.uint32)[: off[-1]]
    dense = np.zeros((H * W, N), dtype=np.int32)
    dense[pix, k] = cost
    ref = lfo.sgm(dense.reshape(H, W, N), P1, P2, npaths, lo=lo, hi=hi).reshape(H * W, N)
    assert np.array_equal(got.astype(np.int64), ref[pix, k].astype(np.int64))
    return int(ws[12:16].view(torch.int32))


@pytest.mark.parametrize("H,W,N,npaths,widths,share,four", [
    (290, 301, 100, 16, [7], None, 1),
    (301, 290, 100, 16, [7, 100], 0.12, 1),
    (290, 301, 100, 16, [21], None, 0),
    (290, 301, 128, 16, [128], None, 1),
    (290, 301, 64, 16, [64], None, 0),
    (290, 301, 40, 16, [5, 40], 0.1, 1),
    (290, 301, 40, 16, [5, 40], 0.8, 0),
    (290, 301, 14, 16, [14], None, 1),            # never wide
    (520, 516, 96, 16, [15], None, 0),            # 8,256
    (520, 516, 64, 16, [7, 64], 0.3, 1),
    (536, 540, 96, 16, [15], None, 0),            # 8,576
    (536, 540, 96, 16, [33], None, 1),
    (301, 300, 200, 8, [9], None, 1),
    (301, 300, 200, 8, [21], None, 0),
    (301, 300, 150, 8, [9, 150], 0.1, 1),
    (301, 300, 150, 8, [40], None, 0),
    (301, 300, 256, 8, [256], None, 1),
    (281, 300, 100, 16, [7], None, 0),            # 4,496: one line per wave always
    (287, 300, 200, 8, [7], None, 0),             # 2,296
])
def test_choice(H, W, N, npaths, widths, share, four):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert _run(H, W, N, npaths, 32, 17, 35, widths, share) == four


@pytest.mark.parametrize("H,W,N,npaths,sum_bits,P1,P2,widths", [
    (690, 701, 100, 16, 32, 17, 35, [7, 7, 7, 100]),
    (701, 690, 70, 16, 16, 17, 35, [1, 7, 13, 14, 15, 16, 17, 70]),
    (693, 690, 64, 16, 32, 6, 48, [3, 14, 64]),
    (690, 691, 33, 16, 32, 6, 16000, [15, 16, 33]),
    (566, 571, 255, 16, 32, 17, 35, [7, 40, 250, 255]),
    (571, 566, 256, 16, 16, 9, 35, [9, 13, 256]),
    (1003, 1005, 160, 16, 32, 17, 35, [7, 15]),
])
def test_four_lines_of_any_ranges(H, W, N, npaths, sum_bits, P1, P2, widths):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert _run(H, W, N, npaths, sum_bits, P1, P2, widths) == 1


def test_choice_in_a_batch():
    # narrow and wide windows, and none, in one plan: each light field takes its own form
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as lfo
    from paper_1907_13449_amd import lf
    lfo.build(force=False)
    items, refs = [], []
    for seed, (H, W, N, lam) in enumerate([(190, 203, 60, 2), (199, 187, 90, 12),
                                           (180, 190, 40, -1), (160, 150, 200, 9)]):
        lfd = lfsynth.workload("paper_s", seed=seed + 50, H=H, W=W, S=3, T=3, N=N)
        p = dict(lfd.params, lam=lam, npaths=16, sum_bits=32)
        refs.append(lfo.depth(lfd.views, lfd.hyp, p))
        items.append((torch.from_numpy(lfd.views).cuda(), torch.from_numpy(lfd.hyp).cuda(), p,
                      torch.empty((H, W), device="cuda"),
                      torch.empty((H, W), dtype=torch.int16, device="cuda")))
    plan = lf.Plan(items)
    plan.capture()
    for rep in range(3):
        for it in items:
            it[3].fill_(float("nan"))
            it[4].fill_(-7)
        torch.cuda.synchronize()
        print("choice in a batch, replay", rep, flush=True)
        plan.run()
        torch.cuda.synchronize()
        for it, ref in zip(items, refs):
            assert np.array_equal(it[4].cpu().numpy(), ref["d_index"])
            assert np.array_equal(it[3].cpu().numpy(), ref["disparity"])
