"""Bins split over workgroups (re-weighting and exit ranges) at the edges of
the split: 1 exit, one workgroup's stride, the smallest part and one more, a
remainder, flagged exits at a bin's start; against numpy over the plan's own
exit records.  Sums of at most 2e4 FP64 terms: 1e-12 for the mean, 1e-9 for
the standard error (the variance of weights about one of them loses at most N
ulps)."""
import numpy as np
import pytest

from paper_2502_06319_amd import workloads as W

pytestmark = pytest.mark.gpu


def _check(plan, job, n_lis, n_knots, n_hist):
    plan.execute()
    ex = plan.read(exits=True)[0]["exits"]
    rng = np.random.default_rng(n_lis)
    lnP0, dlnP = -2.0, 8.0 / n_knots
    x = lnP0 + dlnP * np.arange(n_knots)
    rows = rng.uniform(8, 10, (n_lis, 1)) - rng.uniform(2.3, 3.3, (n_lis, 1)) * x
    flux, se = plan.reweight(lnP0, dlnP, rows)
    pm, hist = plan.exit_range(n_hist)
    at = 0
    for b, (P0, n) in enumerate(zip(job["rigidity_gv"], job["particles_per_bin"])):
        P = ex["P"][at:at + n][ex["flags"][at:at + n] == 0]
        at += n
        if len(P) == 0:
            assert pm[b] == 0 and np.all(flux[:, b] == 0) and np.all(se[:, b] == 0)
            assert hist[b].sum() == 0
            continue
        y = (np.log(P) - lnP0) / dlnP
        k = np.clip(np.floor(y), 0, n_knots - 2).astype(int)
        w = np.exp(rows[:, k] + (y - k) * (rows[:, k + 1] - rows[:, k])) * (P0 / P) ** 2
        np.testing.assert_allclose(flux[:, b], w.mean(1), rtol=1e-12)
        if len(P) > 1:
            np.testing.assert_allclose(se[:, b], w.std(1, ddof=1) / np.sqrt(len(P)), rtol=1e-9)
        assert pm[b] == P.max() and hist[b].sum() == len(P)


@pytest.mark.parametrize("counts", [[1, 255, 1024], [1025, 4097, 2], [256, 20001, 4096]])
@pytest.mark.parametrize("n_lis,n_knots,n_hist", [(1, 2, 1), (17, 40, 4096), (16, 256, 129)])
def test_split_bins_against_numpy(eng, counts, n_lis, n_knots, n_hist):
    job = W.make_job(W.helio_1d(), W.species("p"), [0.7, 2.0, 9.0], counts)
    for cap in (10_000_000, 500):  # 500 steps: about half of the exits are capped
        job["step_cap"] = cap
        plan = eng.plan(job, "mixed", exits=True)
        _check(plan, job, n_lis, n_knots, n_hist)
        plan.destroy()


def test_split_bins_of_equal_weights(eng):
    """No wind: every weight of a bin is the same, its standard error 0."""
    h = W.helio_1d(v=0.0)
    plan = eng.plan(W.make_job(h, W.species("p"), [1.0, 4.0], [9000, 3]), "fp64")
    plan.execute()
    plan.read()
    flux, se = plan.reweight(0.0, 0.5, np.tile(np.linspace(9.0, -9.0, 13), (5, 1)))
    plan.destroy()
    np.testing.assert_array_equal(se, 0.0)
    np.testing.assert_allclose(flux, np.tile([np.exp(9.0), np.exp(9.0 - 1.5 * np.log(4.0) / 0.5)],
                                             (5, 1)), rtol=1e-12)
