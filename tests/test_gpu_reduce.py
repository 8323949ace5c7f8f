"""The per-bin reduction where its sums, its time or its memory could go wrong:
standard errors of bins whose first exit is far from the mean, bins whose exits
are nearly all capped, bins of very different sizes."""
import time

import numpy as np
import pytest

from paper_2502_06319_amd import cosmica as C
from paper_2502_06319_amd import workloads as W

pytestmark = pytest.mark.gpu

LD = np.longdouble


def _reduce_ms(eng, job, precision="mixed"):
    """Shortest of four reductions of the job, ms."""
    plan = eng.plan(job, precision)
    ms = []
    for _ in range(4):
        plan.execute()
        ms.append(eng.timings()["reduce_ms"])
    plan.destroy()
    return min(ms)


@pytest.mark.parametrize("bins,per_bin", [(1100, 300), (1000, 1100)])
def test_standard_error_does_not_depend_on_the_first_exit(eng, bins, per_bin):
    """A steep spectrum, so that a few exits of a bin hold most of its weight;
    in some bins the first exit is one of them, z standard deviations from the
    mean.  The weight of an exit carries at most 2.5 ulps and each sum of the
    two passes a dozen roundings: 16 units of 2^-53, on the standard error
    times the weights' size over their spread (an error that grows with z^2
    would reach 1e-14 here).  One workgroup per bin, and one per part."""
    sp = dict(W.species("p"), lis_index=-10.0)
    job = W.make_job(W.helio_1d(), sp, [1.0] * bins, [per_bin] * bins, seed=5)
    r = eng.run(job, "fp64", exits=True)[0]
    P = r["exits"]["P"].reshape(bins, per_bin).astype(LD)
    w = LD(sp["lis_norm"]) * P ** LD(8.0)
    mean = w.mean(1)
    m2 = ((w - mean[:, None]) ** 2).sum(1)
    z2 = (w[:, 0] - mean) ** 2 / (m2 / per_bin)
    assert z2.max() > 50
    se = np.sqrt(m2 / (per_bin - 1) / per_bin)
    u = LD(2.0) ** -53
    np.testing.assert_array_less(np.abs(r["flux"] / mean - 1), 16 * u)
    np.testing.assert_array_less(np.abs(r["flux_se"] / se - 1),
                                 16 * u * np.sqrt(1 + per_bin * mean**2 / m2))


def test_capped_exits_cost_no_more_than_others(eng):
    """2,000,000 exits of one bin: all capped, and none."""
    job = W.make_job(W.helio_1d(), W.species("p"), [2.0], [2_000_000])
    full = _reduce_ms(eng, job)
    assert _reduce_ms(eng, dict(job, step_cap=1)) < 1.5 * full + 0.05


def test_memory_follows_the_exits_of_each_bin():
    """1,000 bins of 50 exits and one of 600,000: the plan holds 20 B an exit,
    its tables and results, and a few bytes for the parts of each bin."""
    job = W.make_job(W.helio_1d(), W.species("p"), [2.0] * 1001, [50] * 1000 + [600_000])
    with C.Engine(0) as e:
        before = e.serve_stats()["bytes_in_use"]
        plan = e.plan(job, "mixed")
        held = e.serve_stats()["bytes_in_use"] - before
        plan.destroy()
    assert held < 1.25 * 20 * 650_000


@pytest.mark.parametrize("small,large", [([], [4_194_304, 4_300_000]),
                                         ([50], [600_000, 600_000])])
def test_one_large_bin_is_spread(eng, small, large):
    """A bin just past 2^22 exits takes about as long as one of 2^22, and a large
    one among 1,100 small ones as long as among 1,000."""
    ms = []
    for n_small, n in zip((1000, 1100), large):
        counts = small * n_small + [n]
        job = W.make_job(W.helio_1d(), W.species("p"), [2.0] * len(counts), counts)
        ms.append(_reduce_ms(eng, job))
    assert ms[1] < 1.5 * ms[0] + 0.05


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_a_workgroup_per_bin_and_per_part_give_the_same_bits(eng, precision):
    """Bins at the edges of the parts, alone (spread) and among 5,000 one-exit
    bins, where a workgroup takes a whole bin."""
    counts = [1, 1023, 1024, 1025, 2048, 3073, 7000]
    job = W.make_job(W.helio_1d(), W.species("p"), W.log_bins(0.5, 20.0, len(counts)), counts)
    many = [dict(job, rigidity_gv=[3.0] * 500, particles_per_bin=[1] * 500, job_tag=i + 1)
            for i in range(10)]
    for cap in (10_000_000, 500):
        job["step_cap"] = cap
        alone = eng.run(job, precision)[0]
        among = eng.run([job] + many, precision)[0]
        for k in among:
            np.testing.assert_array_equal(alone[k], among[k], err_msg=k)


def test_more_parts_than_a_group(eng):
    """300,000 and 262,145 exits: two groups of parts, against 64-bit two-pass
    sums of the exit records (the weights' 2.5 ulps and a few more for the
    sums: 16 units of 2^-53, on the standard error times sqrt(1 + n mean^2 /
    m2))."""
    counts = [300_000, 262_145]
    job = W.make_job(W.helio_1d(), W.species("p"), [1.0, 4.0], counts)
    r = eng.run(job, "mixed", exits=True)[0]
    at = 0
    for b, (P0, n) in enumerate(zip(job["rigidity_gv"], counts)):
        ex = r["exits"][at:at + n]
        at += n
        w = LD(W.LIS_NORM) * ex["P"].astype(LD) ** LD(-W.LIS_INDEX - 2.0) * LD(P0) ** 2
        m2 = ((w - w.mean()) ** 2).sum()
        u = LD(2.0) ** -53
        assert abs(r["flux"][b] / w.mean() - 1) < 16 * u
        assert abs(r["flux_se"][b] / np.sqrt(m2 / (n - 1) / n) - 1) < (
            16 * u * np.sqrt(1 + n * w.mean() ** 2 / m2))
        assert r["hist"][b].sum() == n and r["steps"][b] == ex["n"].sum()


@pytest.mark.parametrize("bins,per_bin,seed,z2_least", [(1100, 300, 4, 280), (200, 5000, 14, 2900)])
def test_reweighted_standard_error_does_not_depend_on_the_first_exit(eng, bins, per_bin, seed,
                                                                     z2_least):
    """As above for tabulated spectra, whole bins and split ones.  ln J = 8 ln P
    from two knots 4 apart in ln P: with ln P < 2.8 the logarithm, the position
    and the interpolation leave 8e-15 in the exponent, 72 units of 2^-53; 128
    with the exponential and the sums."""
    job = W.make_job(W.helio_1d(), W.species("p"), [1.0] * bins, [per_bin] * bins, seed=seed)
    plan = eng.plan(job, "fp64", exits=True)
    plan.execute()
    P = plan.read(exits=True)[0]["exits"]["P"].reshape(bins, per_bin).astype(LD)
    flux, se = plan.reweight(0.0, 4.0, [[0.0, 32.0]])
    plan.destroy()
    w = P ** LD(6.0)
    mean = w.mean(1)
    m2 = ((w - mean[:, None]) ** 2).sum(1)
    assert ((w[:, 0] - mean) ** 2 / (m2 / per_bin)).max() > z2_least
    u = LD(2.0) ** -53
    np.testing.assert_array_less(np.abs(flux[0] / mean - 1), 128 * u)
    np.testing.assert_array_less(np.abs(se[0] / np.sqrt(m2 / (per_bin - 1) / per_bin) - 1),
                                 128 * u * np.sqrt(1 + per_bin * mean**2 / m2))


def test_reweighting_of_capped_exits_costs_no_more_than_of_others(eng):
    """16 spectra over 2,000,000 exits of one bin: all capped, and none."""
    ms = []
    for cap in (0, 1):
        job = W.make_job(W.helio_1d(), W.species("p"), [2.0], [2_000_000])
        job["step_cap"] = cap
        plan = eng.plan(job, "mixed")
        plan.execute()
        plan.read()
        t = []
        for _ in range(4):
            t0 = time.perf_counter()
            plan.reweight(-3.0, 0.25, np.zeros((16, 40)))
            t.append(1e3 * (time.perf_counter() - t0))
        plan.destroy()
        ms.append(min(t))
    assert ms[1] < 1.5 * ms[0] + 0.2


@pytest.mark.parametrize("counts", [[255, 256, 257, 1], [65536, 65537, 131073, 5]])
def test_reweighting_at_the_edges_of_its_parts(eng, counts):
    """Flagged exits at a part's start (half of the exits capped) and parts of
    2^16 among so many spectra that whole bins would fill the device."""
    n_lis = 4096 if max(counts) > 1000 else 17
    job = W.make_job(W.helio_1d(), W.species("p"), [0.7, 2.0, 9.0, 3.0], counts)
    rng = np.random.default_rng(1)
    x = -2.0 + 0.5 * np.arange(17)
    rows = rng.uniform(8, 10, (n_lis, 1)) - rng.uniform(2.3, 3.3, (n_lis, 1)) * x
    for cap in (0, 500):
        job["step_cap"] = cap
        plan = eng.plan(job, "mixed", exits=True)
        plan.execute()
        ex = plan.read(exits=True)[0]["exits"]
        flux, se = plan.reweight(-2.0, 0.5, rows)
        plan.destroy()
        at = 0
        for b, (P0, n) in enumerate(zip(job["rigidity_gv"], counts)):
            e = ex[at:at + n]
            at += n
            P = e["P"][e["flags"] == 0]
            if len(P) < 2:
                continue
            for l in (0, n_lis - 1):
                # a power law: exact between the knots
                g = (rows[l, 0] - rows[l, -1]) / 8.0
                w = np.exp(rows[l, 0] - g * (np.log(P) + 2.0)) * (P0 / P) ** 2
                np.testing.assert_allclose(flux[l, b], w.mean(), rtol=1e-12)
                np.testing.assert_allclose(se[l, b], w.std(ddof=1) / np.sqrt(len(P)), rtol=1e-12)


def test_static_array_filled_to_its_limit(eng):
    """The largest bin that cosmica_run_static takes (to 64 exits) is spread
    over workgroups too, in about the time of a plan's reduction and with the
    same bits."""
    job = W.make_job(W.helio_1d(), W.species("p"), [2.0], [1])
    job["step_cap"] = 40
    lo, hi = 6_000_000, 7_000_000
    while hi - lo > 64:
        n = (lo + hi) // 2
        try:
            got = eng.run_static(dict(job, particles_per_bin=[n]), "mixed")[0]
            lo = n
        except C.CosmicaError as err:
            assert err.status == C.ESCRATCH
            hi = n
    job["particles_per_bin"] = [lo]
    ms = []
    for _ in range(4):
        got = eng.run_static(job, "mixed")[0]
        ms.append(eng.timings()["reduce_ms"])
    want = eng.run(job, "mixed")[0]
    for k in want:
        np.testing.assert_array_equal(got[k], want[k], err_msg=k)
    assert min(ms) < 1.5 * _reduce_ms(eng, job) + 0.05
