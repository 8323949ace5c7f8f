"""Which kernel a pass and a served slice run: the launch of the rule's choice,
the latency kernel's where it is its, and results that do not depend on it."""
import numpy as np
import pytest

from paper_2502_06319_amd import cosmica as C
from paper_2502_06319_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("hist", "flux", "flux_se", "mean_exit_time_s", "steps", "n_capped", "n_nan")
WAVES = 1024


def _job(model, n, **kw):
    if model == 0:
        job = W.make_job(W.helio_1d(), W.species("p"), [2.0], [n])
    else:
        job = W.make_job(W.c2_helio(), W.species("p"), [2.0], [n])
    job.update(kw)
    return job


def _same(a, b):
    for k in KEYS:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("n", [1, 65, WAVES, WAVES + 1, 16 * WAVES, 64 * WAVES, 64 * WAVES + 1])
def test_small_passes_run_the_latency_kernel(model, precision, n):
    """By default, in as many workgroups as spread the particles over 1,024 waves
    (1,025 particles: 2 a wave, 8 a workgroup, 129 of them); in a set shape
    never, and with the same bits."""
    job = _job(model, n, step_cap=200)
    with C.Engine(0) as e:
        few = e.run(job, precision)[0]
        assert e.passes()["latency"][model] == 1
        assert e.passes()["latency"][1 - model] == 0
        per_wave = min(64, -(-n // WAVES))
        if n <= 64 * WAVES:
            assert e.timings()["grid_blocks"] == -(-n // (4 * per_wave))
        e.set_launch(model, precision, block=256, blocks_per_cu=0, chunk=32, order=2)
        full = e.run(job, precision)[0]
        assert e.passes() == {"latency": (0, 0), "handed_over": 0, "slices": 0, "latency_slices": 0}
        assert e.timings()["grid_blocks"] == -(-n // 256)
    _same(few, full)


@pytest.mark.parametrize("precision,energy", [("mixed", 0), ("mixed", 1), ("fp64", 0)])
def test_particles_are_handed_over(precision, energy):
    """A pass with more than twice as many particles as lanes and paths along the
    sheet hands some over: at most one a lane, and not in run_static, whose
    results are the same.  (The cap lets exits come first, so that the lanes of
    a wave hold particles of different ages when the queue is empty.)"""
    job = W.make_job(W.c2_helio(), W.species("e-"), W.log_bins(0.3, 30.0, 10), 6000, seed=21)
    job.update(step_cap=5000, formulation=energy)
    with C.Engine(0) as e:
        e.set_launch(1, precision, block=64, blocks_per_cu=1)
        got = e.run(job, precision)[0]
        lanes = e.timings()["grid_blocks"] * 64
        p = e.passes()
        assert 60_000 >= 2 * lanes
        assert 0 < p["handed_over"] <= lanes and p["latency"] == (0, 0)
        want = e.run_static(job, precision)[0]
        assert e.passes()["handed_over"] == 0
    _same(got, want)


@pytest.mark.parametrize("explicit", [False, True])
def test_served_slices_are_counted_by_kernel(explicit):
    """One small request: every slice in the latency kernel, or none in a set
    shape."""
    job = _job(1, 3000)
    with C.Engine(0) as e:
        if explicit:
            e.set_launch(1, "mixed")
        t = e.submit(job, "mixed")
        assert t.wait(60000) == C.OK
        p = e.passes()
        _same(t.result(), e.run(job, "mixed")[0])
    assert p["slices"] > 0
    assert p["latency_slices"] == (0 if explicit else p["slices"])


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_the_choice_of_the_launch_can_be_returned(precision):
    """A shape read, changed and set back stays set; reset_launch returns to the
    library's choice, for passes and served slices."""
    job = _job(1, 2000, step_cap=300)
    with C.Engine(0) as e:
        want = e.run(job, precision)[0]
        assert e.passes()["latency"] == (0, 1)
        shape = e.get_launch(1, precision)
        for block in (64, 256):
            e.set_launch(1, precision, **dict(shape, block=block))
            _same(e.run(job, precision)[0], want)
            assert e.passes()["latency"] == (0, 0)
        assert e.get_launch(1, precision) == shape
        e.reset_launch(1, precision)
        assert e.get_launch(1, precision) == shape
        _same(e.run(job, precision)[0], want)
        assert e.passes()["latency"] == (0, 1)
        t = e.submit(job, precision)
        assert t.wait(60000) in (C.OK, C.ESTEPCAP)
        _same(t.result(), want)
        p = e.passes()
        assert p["latency_slices"] == p["slices"] > 0
        for bad in ((2, 0), (0, 2), (-1, 0)):
            assert C.load().cosmica_reset_launch(e.handle, *bad) == C.EINVAL


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_the_default_launch_changes_no_bit_of_a_mixed_batch(eng, precision):
    """Both models in one batch, of several sizes, by default and in set shapes."""
    jobs = [_job(1, 700, job_tag=1), _job(0, 65, job_tag=2), _job(1, 17 * WAVES, job_tag=3)]
    want = eng.run(jobs, precision)
    assert eng.passes()["latency"] == (1, 1)
    for shape in ((256, 0, 32, 2), (64, 1, 1, 1), (128, 2, 1024, 0)):
        for model in (0, 1):
            eng.set_launch(model, precision, *shape)
        for a, b in zip(eng.run(jobs, precision), want):
            _same(a, b)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("block,per_cu,chunk", [(256, 4, 32), (128, 2, 1024), (64, 1, 1)])
def test_a_tuned_context_picks_the_kernel_too(tmp_path, precision, block, per_cu, chunk):
    """The tuner's shape (from its cache here) is the throughput kernel's: small
    passes and served slices run the latency kernel as without it, large ones
    the tuned shape, all with the bits of a context that was not tuned."""
    small = _job(1, 2000, step_cap=300)
    large = _job(1, 6_000_000, step_cap=20)
    cache = tmp_path / "tuned.txt"
    with C.Engine(0) as e:
        want, want_large = e.run(small, precision)[0], e.run(large, precision)[0]
        assert e.passes()["latency"] == (0, 0)
    key = next(l.split()[0] for l in open(_cache_of(tmp_path)))
    cache.write_text("%s 1 %d %d %d %d 2 1e10\n" % (key, C.PRECISION[precision], block, per_cu, chunk))
    with C.Engine(0) as e:
        cfg = e.tune(1, precision, str(cache))
        assert cfg == {"block": block, "blocks_per_cu": per_cu, "chunk": chunk, "order": 2}
        _same(e.run(small, precision)[0], want)
        assert e.passes()["latency"] == (0, 1) and e.timings()["block"] == 256
        _same(e.run_static(small, precision)[0], want)
        assert e.passes()["latency"] == (0, 1)
        _same(e.run(large, precision)[0], want_large)
        assert e.passes()["latency"] == (0, 0)
        assert e.timings()["block"] == block
        assert e.timings()["grid_blocks"] * block <= 64 * WAVES * per_cu
        t = e.submit(small, precision)
        assert t.wait(60000) in (C.OK, C.ESTEPCAP)
        _same(t.result(), want)
        p = e.passes()
        assert p["latency_slices"] == p["slices"] > 0
        e.set_launch(1, precision, **cfg)  # a caller's shape is used for all
        _same(e.run(small, precision)[0], want)
        assert e.passes()["latency"] == (0, 0)


def _cache_of(tmp_path):
    """A tuner cache that names this library's key (a sweep of the radial model)."""
    path = tmp_path / "key.txt"
    with C.Engine(0) as e:
        e.tune(0, "mixed", str(path))
    return path


def test_small_requests_together_run_the_latency_kernel(monkeypatch):
    """Eight requests of 1,000 particles, cut to chunks of one: far fewer than
    the 131,072 lanes up to which slices run the latency kernel; in slices that
    park and resume many times."""
    monkeypatch.setenv("COSMICA_SLICE_MS", "0.2")
    jobs = [W.make_job(W.c2_helio(), W.species("p"), W.log_bins(0.3, 30.0, 20), 50, seed=3 + i,
                       job_tag=i) for i in range(8)]
    with C.Engine(0) as e:
        tickets = [e.submit(j, "mixed") for j in jobs]
        for t in tickets:
            assert t.wait(60000) == C.OK
        p = e.passes()
        for j, t in zip(jobs, tickets):
            _same(t.result(), e.run(j, "mixed")[0])
    assert p["latency_slices"] == p["slices"] > 2


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_a_plan_laid_out_before_a_shape_is_set(precision):
    """Its queue has chunks of one particle, for the latency kernel (0.36 ms in the
    throughput kernel, 0.32 with chunks of 32): the first execution in a set
    shape cuts one of 2 x 500 / 32 chunks of 16 B, once; back in the default
    shape it runs the latency kernel.  Always the same bits."""
    job = W.make_job(W.helio_1d(), W.species("p"), [2.0, 9.0], [500, 500])
    with C.Engine(0) as e:
        plan = e.plan(job, precision)
        plan.execute()
        want = plan.read()[0]
        held = e.serve_stats()["bytes_in_use"]
        e.set_launch(0, precision)
        for _ in range(2):
            plan.execute()
            _same(plan.read()[0], want)
            assert e.passes()["latency"] == (0, 0)
            assert e.serve_stats()["bytes_in_use"] - held == 512
        e.reset_launch(0, precision)
        plan.execute()
        _same(plan.read()[0], want)
        assert e.passes()["latency"] == (1, 0)
        plan.destroy()
