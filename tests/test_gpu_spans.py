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


def _by_hand(A, w, n, pad=True):
    """n steps one launch of one step at a time: the schedule from the host
    controller, each sync the one-step fused call."""
    st = A.adpsgd_sched_init(A.hparams_of(w))
    syncs, var = [], []
    with A.Adpsgd.from_workload(w, pad_rows=pad) as eng:
        for _ in range(n):
            t = st.t
            if A.adpsgd_sched_step(eng.hp, st):
                v = eng.step_average()
                A.adpsgd_sched_on_sync(eng.hp, st, t, float(sum(v)))
                syncs.append(t)
                var.append(v)
            else:
                eng.local_steps(1)
        return eng.x.cpu().numpy(), eng.m.cpu().numpy(), syncs, np.asarray(var)


# worker counts of every layout: compiled (one row per wave, and several with
# enough chunks), K an argument with 1, 2, 4 and 8 rows per wave (whole and
# ragged last waves), the loop kernel; the larger sizes give the layouts of more
# rows per wave two waves per SIMD, just, 3,000 elements none
@pytest.mark.parametrize("avg_m", [False, True])
@pytest.mark.parametrize("K,P", [(1, 3000), (2, 530_001), (4, 270_001), (8, 140_001), (16, 140_001), (32, 70_001), (8, 3000),
                                 (32, 3000), (4, 524_289), (8, 524_035), (32, 131_073), (3, 9001), (7, 9001), (24, 9001), (25, 9001), (31, 5001), (33, 5001), (48, 5001), (49, 5001),
                                 (64, 5001), (65, 3001),
                                 (100, 3001), (128, 3000), (129, 2001)])
def test_run_equals_one_step_launches(A, K, P, avg_m):
    """A constant-period run (whole spans of syncs) against single-step launches:
    the replicas and momenta bit for bit, the variances to the rounding of
    their sums, with tensors that begin inside a chunk."""
    w = _w(K=K, sizes=(700, 1, 3, 0, 280, P - 984), p_init=3, total_steps=40, avg_momentum=avg_m)
    n = 23
    x, m, syncs, var = _by_hand(A, w, n)
    with A.Adpsgd.from_workload(w) as eng:
        recs, v, _ = eng.run(n)
        assert list(recs["t"]) == syncs
        assert np.array_equal(eng.x.cpu().numpy(), x) and np.array_equal(eng.m.cpu().numpy(), m)
    assert np.allclose(v, var, rtol=1e-12, atol=0.0)


@pytest.mark.parametrize("K,pad", [(4, False), (8, True), (5, False), (100, False)])
def test_unaligned_and_cut_rows(A, K, pad):
    """Packed rows of a length that is not a multiple of 4, and a last chunk cut
    inside a group, in launches of several steps and syncs."""
    w = _w(K=K, sizes=(255, 2, 257, 1301), p_init=2, total_steps=40)
    x, m, syncs, var = _by_hand(A, w, 17, pad)
    with A.Adpsgd.from_workload(w, pad_rows=pad) as eng:
        recs, v, _ = eng.run(17)
        assert np.array_equal(eng.x.cpu().numpy(), x) and np.array_equal(eng.m.cpu().numpy(), m)
    assert list(recs["t"]) == syncs and np.allclose(v, var, rtol=1e-12, atol=0.0)


# rows that start 4, 8 and 12 bytes behind a 16-byte boundary: whole chunks move with
# four-byte aligned vectors, in every layout, and leave the neighbouring rows alone
@pytest.mark.parametrize("P", [2305, 2306, 2307, 140_001])
@pytest.mark.parametrize("K", [1, 2, 3, 4, 7, 8, 16, 25, 32, 48, 64, 100])
def test_whole_chunks_of_unaligned_rows(A, K, P):
    w = _w(K=K, sizes=(1024, P - 1029, 5), p_init=3, total_steps=40, avg_momentum=K % 2 == 0)
    x, m, syncs, var = _by_hand(A, w, 10, False)
    xp, mp, _, _ = _by_hand(A, w, 10, True)
    assert np.array_equal(x, xp) and np.array_equal(m, mp)
    with A.Adpsgd.from_workload(w, pad_rows=False) as eng:
        recs, v, _ = eng.run(10)
        assert np.array_equal(eng.x.cpu().numpy(), x) and np.array_equal(eng.m.cpu().numpy(), m)
    assert list(recs["t"]) == syncs and np.allclose(v, var, rtol=1e-12, atol=0.0)


# periods around the most steps (64) and measurements (16) of a launch; K = 129
# steps one at a time where the device decides
@pytest.mark.parametrize("traced", [False, True])
@pytest.mark.parametrize("K,p,N", [(4, 1, 90), (4, 15, 120), (8, 17, 150), (4, 63, 300), (8, 64, 300), (4, 66, 340),
                                   (8, 130, 500), (129, 3, 40), (129, 1, 40), (200, 9, 90), (160, 70, 300)])
def test_adaptive_periods_agree_under_every_policy(A, K, p, N, traced):
    """Adaptive runs whose period moves (a decisive sync from the second on): the
    default driver's spans, single device-decided steps and host-planned
    spans give the same records and bits."""
    w = _w(K=K, sizes=(2000, 7, 1500), p_init=p, total_steps=N, period_mode=W.PERIOD_ADAPTIVE, k_s=p,
           lr_kind=W.LR_STEP)
    out = []
    for pol in (A.LAUNCH_HYBRID, A.LAUNCH_DEVICE, A.LAUNCH_HOST):
        with A.Adpsgd.from_workload(w) as eng:
            eng.set_launch_policy(pol)
            r = eng.run_traced(N) if traced else eng.run(N)
            st = eng.get_state()
            out.append((r[0].tobytes(), r[1].tobytes(), r[3].tobytes() if traced else b"", eng.x.cpu().numpy().tobytes(),
                        eng.m.cpu().numpy().tobytes(), (st.t, st.cnt, st.p, st.nC2, st.C2)))
    assert len(r[0]) > 1 and out[0] == out[1] == out[2]


# launches of up to 4 and of more measurements whose decisions the device takes (one
# finishing block, or one for each and a kernel for the decisions), on every path of
# the reduction: tensors summed in LDS, in device memory (over 512), in windows
@pytest.mark.parametrize("p", [1, 2, 3, 4, 6])
@pytest.mark.parametrize("sizes", [(2000, 7, 1500), (40,) * 600, (3,) * 3600 + (70_000, 5)])
def test_decisions_of_several_measurements_agree_under_every_policy(A, sizes, p):
    w = _w(K=4, sizes=sizes, p_init=p, total_steps=60, period_mode=W.PERIOD_ADAPTIVE, k_s=2 * p, lr_kind=W.LR_STEP)
    out = []
    for pol in (A.LAUNCH_HYBRID, A.LAUNCH_DEVICE, A.LAUNCH_HOST):
        with A.Adpsgd.from_workload(w) as eng:
            eng.set_launch_policy(pol)
            recs, var, _, steps = eng.run_traced(60)
            st = eng.get_state()
            out.append((recs.tobytes(), var.tobytes(), steps.tobytes(), eng.x.cpu().numpy().tobytes(),
                        (st.t, st.cnt, st.p, st.nC2, st.C2)))
    assert out[0] == out[1] == out[2]


@pytest.mark.parametrize("avg_m", [False, True])
@pytest.mark.parametrize("K,mode,pol", [(4, W.PERIOD_CONST, "HYBRID"), (8, W.PERIOD_ADAPTIVE, "HYBRID"),
                                        (5, W.PERIOD_ADAPTIVE, "HOST"), (16, W.PERIOD_ALG1, "HYBRID")])
def test_rows_are_whole_between_runs(A, K, mode, pol, avg_m):
    """Inside a run the rows behind a sync are kept once.  Runs cut anywhere, at
    a sync, behind one and in a period, with the rows changed by the caller in
    between, equal the same steps launched one by one."""
    w = _w(K=K, sizes=(3000, 5, 600), p_init=3, total_steps=200, avg_momentum=avg_m, period_mode=mode,
           k_s=6 if mode == W.PERIOD_ADAPTIVE else 0)
    cuts = [3, 1, 2, 4, 6, 7, 80, 3]
    with A.Adpsgd.from_workload(w) as a, A.Adpsgd.from_workload(w) as b:
        a.set_launch_policy(getattr(A, "LAUNCH_" + pol))
        for i, n in enumerate(cuts):
            a.run(n)
            st = b.get_state()
            for _ in range(n):
                t = st.t
                if A.adpsgd_sched_step(b.hp, st):
                    v = b.step_average()
                    A.adpsgd_sched_on_sync(b.hp, st, t, float(sum(v)))
                    b.set_state(st)
                else:
                    b.local_steps(1)
            assert np.array_equal(a.x.cpu().numpy(), b.x.cpu().numpy()), (i, n)
            assert np.array_equal(a.m.cpu().numpy(), b.m.cpu().numpy()), (i, n)
            a.x[K - 1].add_(0.01 * (i + 1))       # the caller's own change, to one row
            b.x[K - 1].add_(0.01 * (i + 1))


# periods longer than a launch: one that begins with merged rows and holds no sync, so
# that its waves part ways only at a barrier of its own; blocks of one, several and
# sixteen waves, compiled K and K an argument
@pytest.mark.parametrize("avg_m", [False, True])
@pytest.mark.parametrize("mode", [W.PERIOD_CONST, W.PERIOD_ADAPTIVE])
@pytest.mark.parametrize("K,P", [(2, 3000), (4, 3507), (8, 3507), (8, 600_000), (16, 3507), (16, 140_001), (32, 3507),
                                 (5, 3507), (3, 3507), (100, 2001)])
def test_merged_rows_without_a_sync_in_the_launch(A, K, P, mode, avg_m):
    w = _w(K=K, sizes=(700, 3, P - 703), p_init=130, total_steps=300, avg_momentum=avg_m, period_mode=mode, k_s=100)
    n = 290                                    # two syncs, at 129 and about 259
    x, m, syncs, var = _by_hand(A, w, n)
    assert len(syncs) == 2
    with A.Adpsgd.from_workload(w) as eng:
        recs, v, _ = eng.run(n)
        assert list(recs["t"]) == syncs
        assert np.array_equal(eng.x.cpu().numpy(), x) and np.array_equal(eng.m.cpu().numpy(), m)
    assert np.allclose(v, var, rtol=1e-12, atol=0.0)


def test_rows_are_whole_after_a_failed_sync(A):
    """A run that a non-finite S stops behind a sync leaves whole rows."""
    w = _w(K=4, sizes=(3000, 5), lr_kind=W.LR_CONST, lr0=50.0, p_init=2, total_steps=300, period_mode=W.PERIOD_ADAPTIVE)
    with A.Adpsgd.from_workload(w) as eng:
        with pytest.raises(A.AdpsgdError) as e:
            eng.run(300)
        assert e.value.code == A.ENONFINITE
        st = eng.get_state()
        x = eng.x.cpu().numpy()
    assert st.cnt == 0 and st.t < 300          # stopped behind a sync
    assert all(np.array_equal(x[k], x[0], equal_nan=True) for k in range(4))
