"""Schedules of batch plans: what the defaults come to.  None changes a result."""
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


def test_default_cells_per_thread(lf):
    # four above 2^26 cells, as for one light field, unless told otherwise
    few = _items(lf, [(40, 50, 20), (30, 30, 150)])
    assert _plan(lf, few).tuning["cost_cells_per_thread"] == 2
    large = _items(lf, [(520, 516, 256)], S=3, T=1)
    assert _plan(lf, large).tuning["cost_cells_per_thread"] == 4
    assert _plan(lf, large, dict(cost_cells_per_thread=2)).tuning["cost_cells_per_thread"] == 2
