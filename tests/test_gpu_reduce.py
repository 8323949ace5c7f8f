"""The per-bin reduction where its sums or its time could go wrong: standard
errors of bins whose first exit is far from the mean, bins whose exits are
nearly all capped."""
import numpy as np
import pytest

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
