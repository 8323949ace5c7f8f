"""The latency kernel (few waves per SIMD, random numbers drawn ahead on idle
lanes) against the throughput kernel: results and exit records equal bit for
bit.  An explicit launch shape selects the throughput kernel, the default shape
the latency kernel for passes of this size.  Sizes sit at the edges of its
rules: 1,024 waves at one wave per SIMD, 16 particles per wave (random numbers
ahead), 64 lanes, and the second wave per SIMD."""
import numpy as np
import pytest

from paper_2502_06319_amd import cosmica as C
from paper_2502_06319_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("hist", "flux", "flux_se", "mean_exit_time_s", "steps", "n_capped", "n_nan")
WAVES = 1024


def _both(jobs, precision, model=1):
    """The same call with the latency and with the throughput kernel."""
    with C.Engine(0) as e:
        few = e.run(jobs, precision, exits=True)
        shape = e.timings()
        e.set_launch(model, precision, block=256, blocks_per_cu=0, chunk=32, order=2)
        full = e.run(jobs, precision, exits=True)
    for a, b in zip(few, full):
        for k in KEYS:
            np.testing.assert_array_equal(a[k], b[k], err_msg=k)
        for k in C.EXIT_DTYPE.names:  # field by field: NaN equals NaN
            np.testing.assert_array_equal(a["exits"][k], b["exits"][k], err_msg=k)
    return few, shape


def _job(kind, bins, per_bin, seed=42, tag=0):
    if kind == "radial":
        job = W.c1_job(particles_per_bin=1, seed=seed)
        rig = W.log_bins(0.5, 20.0, bins)
    else:
        job = W.c2_heliosheath_job(1, seed) if kind == "heliosheath" else W.c2_job(1, seed)
        rig = W.log_bins(0.3, 30.0, bins)
    job.update(rigidity_gv=rig, particles_per_bin=[per_bin] * bins, job_tag=tag)
    if kind in ("energy", "energy orbit"):
        job["formulation"] = 1
    if kind == "energy orbit":
        job = W.with_orbit(job, W.ulysses_like_orbit(5))
    return job


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind,n", [("radial", 1), ("radial", 65), ("radial", 17 * WAVES + 3),
                                    ("radial", 64 * WAVES + 1), ("3d", 1), ("3d", WAVES),
                                    ("3d", WAVES + 1), ("3d", 16 * WAVES), ("3d", 16 * WAVES + 1),
                                    ("3d", 64 * WAVES), ("3d", 64 * WAVES + 1),
                                    ("heliosheath", 333), ("heliosheath", 20 * WAVES + 7),
                                    ("energy", 3 * WAVES), ("energy orbit", 33 * WAVES)])
def test_latency_kernel_equals_throughput_kernel(kind, n, precision):
    first = min(n, 7)
    job = _job(kind, 3 if n > 100 else 1, first)
    if n > 100:
        job["particles_per_bin"] = [first, n - first - 5, 5]
    else:
        job["particles_per_bin"] = [n]
    r, shape = _both(job, precision, 0 if kind == "radial" else 1)
    assert int(r[0]["hist"].sum()) == n
    assert shape["grid_blocks"] * shape["block"] <= 3 * 64 * WAVES


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_latency_kernel_mixed_jobs_caps_and_non_finite(precision):
    """Jobs with their own seeds, shapes and formulations in one wave; a step
    cap inside a batch of drawn-ahead numbers; particles that turn non-finite;
    particles that ride the current sheet (phi past a turn, poles, reflections
    through the origin)."""
    sheet = W.make_job(W.c2_helio(), W.species("e-"), [0.5, 5.0], 300, seed=3, job_tag=9)
    sheet["step_cap"] = 3001
    jobs = [_job("3d", 4, 50, seed=5, tag=1), _job("heliosheath", 3, 61, seed=6, tag=2),
            _job("energy", 2, 33, seed=7, tag=3), _job("energy orbit", 2, 40, seed=8, tag=4),
            dict(_job("3d", 2, 70, seed=9, tag=5), step_cap=7), sheet,
            dict(_job("3d", 2, 9, seed=9, tag=6), rigidity_gv=[1.0, 1e20])]
    r, _ = _both(jobs, precision)
    assert np.all(r[4]["n_capped"] == 70)
    assert r[5]["n_capped"].sum() > 0


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("explicit", [False, True])
def test_served_slices_of_both_kernels(precision, explicit, monkeypatch):
    """Requests too small for one particle a wave, of one chunk remainder, and
    of both models, in slices short enough to park and resume many times, with
    the latency kernel's slices (default shape) and without (explicit shape)."""
    monkeypatch.setenv("COSMICA_SLICE_MS", "0.3")
    jobs = [dict(_job("3d", 3, 7, seed=11, tag=1)), dict(_job("energy", 2, 700, seed=12, tag=2)),
            dict(_job("heliosheath", 4, 411, seed=13, tag=3)), dict(_job("radial", 2, 33, seed=14)),
            W.make_job(W.c2_helio(), W.species("e-"), [0.5, 5.0], 100, seed=3, job_tag=9)]
    with C.Engine(0) as e:
        if explicit:
            for m in (0, 1):
                e.set_launch(m, precision)
        tickets = [e.submit(j, precision) for j in jobs]
        for t in tickets:
            assert t.wait(120000) == C.OK
        for j, t in zip(jobs, tickets):
            alone, got = e.run(j, precision)[0], t.result()
            for k in KEYS:
                np.testing.assert_array_equal(got[k], alone[k], err_msg=k)


@pytest.mark.parametrize("precision,energy", [("mixed", 0), ("mixed", 1), ("fp64", 0)])
def test_hand_over_to_the_latency_kernel(precision, energy):
    """A pass with more than twice as many particles as lanes and paths along the
    sheet parks its last particles for the latency kernel: the same bits as in
    run_static, which has no list to hand over with.  The cap keeps paths short
    (and caps most of them)."""
    per = 30000
    job = W.make_job(W.c2_helio(), W.species("e-"), W.log_bins(0.3, 30.0, 10), per, seed=21)
    job.update(step_cap=300, formulation=energy)
    extra = dict(_job("heliosheath", 2, 40, seed=22, tag=3), formulation=energy)
    with C.Engine(0) as e:
        e.set_launch(1, precision, block=256, blocks_per_cu=2)
        before = e.serve_stats()["bytes_in_use"]
        got = e.run([job, extra], precision)
        assert e.serve_stats()["bytes_in_use"] > before
        lanes = e.timings()["grid_blocks"] * 256
        assert 10 * per >= 2 * lanes
        want = e.run_static([job, extra], precision)
        again = e.run([job, extra], precision)
        for a, b, c in zip(got, want, again):
            for k in KEYS:
                np.testing.assert_array_equal(a[k], b[k], err_msg=k)
                np.testing.assert_array_equal(c[k], b[k], err_msg=k)
