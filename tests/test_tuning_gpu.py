"""Schedules of batch plans: what the defaults come to, that each form of the bounded SGM can
be asked for, and that the autotuner leaves alone what no kernel of the batch has.  None
changes a result."""
import pytest

import lfsynth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_13449_amd import lf as binding
    return binding


def _items(lf, shapes, S=3, T=3, **p):
    out = []
    for i, (H, W, N) in enumerate(shapes):
        lfd = lfsynth.workload("paper_s", seed=70 + i, H=H, W=W, S=S, T=T, N=N)
        prm = dict(lfd.params, sum_bits=32, **p)
        views, hyp = torch.from_numpy(lfd.views).cuda(), torch.from_numpy(lfd.hyp).cuda()
        idx = torch.empty((H, W), dtype=torch.int16, device="cuda")
        alone = lf.lf_depth(views, hyp, prm, d_index=idx)
        out.append((alone, idx, (views, hyp, prm, torch.empty((H, W), device="cuda"),
                                 torch.empty((H, W), dtype=torch.int16, device="cuda"))))
    return out


def _plan(lf, items, tuning=None):
    plan = lf.Plan([it[2] for it in items], tuning=tuning)
    _check(plan, items)
    return plan


def _check(plan, items):
    for _, _, it in items:
        it[3].fill_(float("nan"))
        it[4].fill_(-7)
    plan.run()
    torch.cuda.synchronize()
    for alone, idx, it in items:
        assert torch.equal(it[3], alone)
        assert torch.equal(it[4], idx)


def test_defaults(lf):
    few = _items(lf, [(40, 50, 20), (30, 30, 150)])
    assert _plan(lf, few).tuning == dict(cost_cells_per_thread=2, cost_stride=1,
                                         dense_prefetch=16, bounded_prefetch=4,
                                         bounded_lanes=64, bounded_offsets=32)
    # 12,000 path steps per step of the longest line take four lines per wave
    many = _items(lf, [(250, 255, 20)] * 6)
    assert _plan(lf, many).tuning["bounded_lanes"] == 16
    # 5,100: the ranges decide
    some = _items(lf, [(213, 213, 20)] * 3)
    assert _plan(lf, some).tuning["bounded_lanes"] == 0
    # four cells per thread above 2^26 cells, as for one light field, unless told otherwise
    large = _items(lf, [(520, 516, 256)], S=3, T=1)
    assert _plan(lf, large).tuning["cost_cells_per_thread"] == 4
    assert _plan(lf, large, dict(cost_cells_per_thread=2)).tuning["cost_cells_per_thread"] == 2


def test_every_form_of_the_bounded_sgm(lf):
    # the one-line form has a launch for its metadata besides
    many = _items(lf, [(250, 255, 20)] * 6)
    four = _plan(lf, many, dict(bounded_lanes=16))
    one = _plan(lf, many, dict(bounded_lanes=64))
    assert one.launches == four.launches + 1
    assert one.tuning["bounded_lanes"] == 64
    few = _items(lf, [(40, 50, 20), (30, 30, 150)])
    for lanes in (16, 32, 64):
        assert _plan(lf, few, dict(bounded_lanes=lanes)).tuning["bounded_lanes"] == lanes
    with pytest.raises(lf.LFError):
        lf.Plan([few[0][2]], tuning=dict(bounded_lanes=8))


def test_autotuner_keeps_what_no_kernel_has(lf):
    # up to 64 hypotheses the initial SGM has no prefetch depth, and without bounds there
    # are neither its stages nor slices of the bounded cost
    items = _items(lf, [(60, 70, 40), (45, 50, 33)])
    plan = _plan(lf, items)
    chosen = plan.autotune(reps=1)
    assert chosen["dense_prefetch"] == 16
    assert chosen["bounded_lanes"] in (16, 64)
    _check(plan, items)
    boundless = _items(lf, [(60, 70, 100)], lam=-1)
    plan = _plan(lf, boundless)
    chosen = plan.autotune(reps=1)
    assert (chosen["dense_prefetch"], chosen["cost_cells_per_thread"],
            chosen["cost_stride"]) == (16, 2, 1)
    _check(plan, boundless)
    # where the ranges decide, that is a third form
    some = _items(lf, [(213, 213, 80)] * 3)
    plan = _plan(lf, some)
    assert plan.autotune(reps=1)["bounded_lanes"] in (0, 16, 64)
    _check(plan, some)
