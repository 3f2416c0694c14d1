"""Launches of several steps: the same bits as the launches of one step they replace."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2007_06134_amd
    return paper_2007_06134_amd


def _w(K=4, sizes=(4099, 1, 8000, 6), **kw):
    d = dict(name="span", K=K, sizes=tuple(sizes), seed=21, sigma=0.1, momentum=0.9, weight_decay=5e-4,
             h_lo=1e-2, h_hi=1.0, lr_kind=W.LR_COSINE, lr0=0.05, total_steps=200,
             period_mode=W.PERIOD_CONST, p_init=4, k_s=0)
    d.update(kw)
    return W.Workload(**d)


# 1 and 2 steps keep the LDS reservation, 3 and more leave it out; 64 fill a launch, 65 and 130 need more
@pytest.mark.parametrize("n", [1, 2, 3, 64, 65, 130])
@pytest.mark.parametrize("sizes,pad", [((4096 * 3,), True), ((4099, 1, 8000, 7), True), ((4099, 1, 8000, 7), False)])
def test_steps_of_one_call_equal_single_steps(A, n, sizes, pad):
    w = _w(K=5, sizes=sizes)
    with A.Adpsgd.from_workload(w, pad_rows=pad) as a, A.Adpsgd.from_workload(w, pad_rows=pad) as b:
        a.set_step_launch(64, 8192, 3)
        a.local_steps(n)
        for _ in range(n):
            b.local_steps(1)
        assert np.array_equal(a.x.cpu().numpy(), b.x.cpu().numpy())
        assert np.array_equal(a.m.cpu().numpy(), b.m.cpu().numpy())
        sa, sb = a.get_state(), b.get_state()
        assert (sa.t, sa.cnt) == (sb.t, sb.cnt) == (n, n)
