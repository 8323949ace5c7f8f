"""Bins split over workgroups (reduction, re-weighting, exit ranges) at the edges of
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


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_reduction_does_not_depend_on_the_split(eng, precision):
    """A few bins at the edges of the reduction's parts (1,024 exits), alone (a
    workgroup per part) and among 1,100 one-particle bins (a workgroup per
    bin): the same bits; and numpy's statistics of the exit records."""
    counts = [1, 1023, 1024, 1025, 2048, 3073, 7000]
    job = W.make_job(W.helio_1d(), W.species("p"), W.log_bins(0.5, 20.0, len(counts)), counts)
    many = [dict(job, rigidity_gv=[3.0] * 55, particles_per_bin=[1] * 55, job_tag=i + 1)
            for i in range(20)]
    for cap in (10_000_000, 500):
        job["step_cap"] = cap
        alone = eng.run(job, precision, exits=True)[0]
        mixed = eng.run([job] + many, precision)[0]
        for k in mixed:
            np.testing.assert_array_equal(alone[k], mixed[k], err_msg=k)
        at = 0
        for b, (P0, n) in enumerate(zip(job["rigidity_gv"], counts)):
            ex = alone["exits"][at:at + n]
            at += n
            P = ex["P"][ex["flags"] == 0]
            w = W.LIS_NORM * P ** -W.LIS_INDEX * (P0 / P) ** 2
            assert alone["steps"][b] == ex["n"].sum() and alone["hist"][b].sum() == len(P)
            assert alone["n_capped"][b] == n - len(P)
            if len(P) > 1:
                np.testing.assert_allclose(alone["flux"][b], w.mean(), rtol=1e-12)
                np.testing.assert_allclose(alone["flux_se"][b], w.std(ddof=1) / np.sqrt(len(P)),
                                           rtol=1e-9)
                np.testing.assert_allclose(alone["mean_exit_time_s"][b],
                                           ex["t"][ex["flags"] == 0].mean(), rtol=1e-12)
