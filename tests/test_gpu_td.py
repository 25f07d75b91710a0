"""Time-dependent rays (moray_td_*) on the GPU, step by step against the
oracle's orc_trace_td on the same seeded inputs, through the C ABI:

* every step's k_ph within 1e-9 (float64 path) or 1e-4 (mixed path) of the
  oracle's wherever it exceeds 1e-6 of its maximum; the photon rate held in
  flight, escaped and absorbed to the same bar; segment, split, escape and
  truncation counts exact in float64; per-step photon bookkeeping
  emitted + held before = absorbed + escaped + truncated + held after;
* a pulse (emission in the first step only) against the oracle's pulse, and
  a root grid with a refined child holding a source;
* c dt_P beyond the box: one step equals moray_trace;
* a pool too small grows (doubling, within the context's HBM budget) and
  the step runs again from the rays in flight before it, with the results of
  a state created large enough; when the budget leaves no room to grow, the
  step fails with MORAY_EQUEUE and leaves the state as it was (a later step
  fails the same way rather than on a broken state); bad arguments are
  rejected.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1012_2865_amd import moray as M
from paper_1012_2865_amd import workloads as W

pytestmark = pytest.mark.gpu


def _np(a):
    return a.detach().cpu().numpy() if hasattr(a, "detach") else np.asarray(a)


def _rel(got, want):
    got, want = _np(got).ravel(), np.asarray(want).ravel()
    if want.max() == 0.0:
        return 0.0, float(np.abs(got).max())
    m = want > 1e-6 * want.max()
    return float(np.max(np.abs(got[m] - want[m]) / want[m])), float(np.max(np.abs(got - want)) / want.max())


def _problem(item=1):
    return W.lognormal_problem(92, item, 20, 2, mean=1e-4)


def _nested_problem(item=6):
    # a thin root with a 2x-refined child holding one of the sources
    p = _problem(item)
    rng = W.rng_for(92, 100 + item, 0)
    child = W.Grid(n_h=(10 ** rng.uniform(-4.5, -3.5, (12, 12, 12))).astype(np.float32),
                   x_hi=rng.uniform(0.5, 1.0, (12, 12, 12)).astype(np.float32),
                   dx_cm=p.grids[0].dx_cm / 2, parent=0, offset=(4, 5, 6))
    p.grids.append(child)
    p.sources = p.sources.copy()
    p.sources[0, :3] = [7.25, 8.5, 9.75]
    return p


def _compare_steps(precision, emits, cdt=4.0, item=1, make=None):
    p = _problem(item) if make is None else make()
    dev = M.problem_to_device(p)
    ctx = M.moray_init(device=0, precision=precision)
    td = None
    fp64 = precision == M.MORAY_FP64
    tol = 1e-9 if fp64 else 1e-4
    try:
        td = M.moray_td_create(ctx, dev, cdt, 1 << 21)
        rays, held_prev = None, 0.0
        for step, emit in enumerate(emits):
            ref, rays = O.trace_td(p, cdt, rays, emit=emit)
            res, held = M.moray_td_step(ctx, td, dev, emit=emit)
            T = ref["totals"]
            rel, absr = 0.0, 0.0
            for q in range(len(p.grids)):
                rq, aq = _rel(res["k_ph"][q], ref["k_ph"][q])
                rel, absr = max(rel, rq), max(absr, aq)
            print(f"[td prec {precision} step {step} emit {emit}] k_ph max rel {rel:.2e}, held {held:.4e} "
                  f"(oracle {ref['held']:.4e}), in flight {len(rays)}, segments {res['segments']}/{T['segments']}",
                  flush=True)
            assert rel <= tol and absr <= max(tol, 1e-6), (step, rel, absr)
            assert held == pytest.approx(ref["held"], rel=tol, abs=1e-12 * max(T["emitted"], held_prev, 1.0))
            for k in ("escaped", "absorbed", "truncated"):
                assert res[k] == pytest.approx(T[k], rel=max(tol, 1e-12), abs=1e-12 * max(T["emitted"], held_prev)), k
            assert res["emitted"] == pytest.approx(T["emitted"], rel=1e-14)
            bal = res["emitted"] + held_prev - res["absorbed"] - res["escaped"] - res["truncated"] - held
            assert abs(bal) <= 1e-9 * max(res["emitted"], held_prev), (step, bal)
            if fp64:
                for k in ("segments", "splits", "rays_escaped", "rays_truncated", "rays_seeded"):
                    assert res[k] == T[k], (step, k, res[k], T[k])
            held_prev = held
    finally:
        if td:
            M.moray_td_free(ctx, td)
        M.moray_free(ctx)


@pytest.mark.parametrize("precision", [M.MORAY_FP64, M.MORAY_FP32_ACC64])
def test_steps_match_the_oracle(precision):
    _compare_steps(precision, [True] * 8)


@pytest.mark.parametrize("precision", [M.MORAY_FP64, M.MORAY_FP32_ACC64])
def test_nested_grids_match_the_oracle(precision):
    _compare_steps(precision, [True] * 5, cdt=5.0, make=_nested_problem)


@pytest.mark.parametrize("precision", [M.MORAY_FP64, M.MORAY_FP32_ACC64])
def test_a_pulse_matches_the_oracle(precision):
    _compare_steps(precision, [True, False, False, False], cdt=3.0, item=2)


def test_infinite_speed_of_light_is_moray_trace():
    p = _problem(3)
    dev = M.problem_to_device(p)
    ctx = M.moray_init(device=0, precision=M.MORAY_FP64)
    try:
        one = M.moray_trace(ctx, [dev])[0]
        td = M.moray_td_create(ctx, dev, 1e6, 1 << 21)
        try:
            res, held = M.moray_td_step(ctx, td, dev)
        finally:
            M.moray_td_free(ctx, td)
    finally:
        M.moray_free(ctx)
    assert held == 0.0
    a, b = _np(res["k_ph"][0]), _np(one["k_ph"][0])
    assert np.allclose(a, b, rtol=1e-12, atol=1e-14 * b.max())
    for k in ("segments", "splits", "rays_escaped", "rays_truncated", "rays_seeded"):
        assert res[k] == one[k], k


def test_overflow_and_bad_arguments():
    p = _problem(4)
    dev = M.problem_to_device(p)
    ctx = M.moray_init(device=0, precision=M.MORAY_FP32_ACC64)
    try:
        for c_dt, pool in ((0.0, 1 << 16), (float("inf"), 1 << 16), (4.0, 100)):
            with pytest.raises(M.MorayError) as e:
                M.moray_td_create(ctx, dev, c_dt, pool)
            assert e.value.status == M.MORAY_EINVAL
        # a context whose HBM budget holds the small state but not a doubled one
        tight = M.moray_init(device=0, precision=M.MORAY_FP32_ACC64, hbm_budget_bytes=2 << 20)
        td = M.moray_td_create(tight, dev, 4.0, 1024)      # far too small for this problem's rays
        try:
            for _ in range(2):
                with pytest.raises(M.MorayError) as e:
                    M.moray_td_step(tight, td, dev)
                assert e.value.status == M.MORAY_EQUEUE
                assert "budget" in str(e.value)
        finally:
            M.moray_td_free(tight, td)
            M.moray_free(tight)
        td = M.moray_td_create(ctx, dev, 4.0, 1 << 16)
        try:
            other = M.problem_to_device(W.lognormal_problem(92, 5, 16, 2, mean=1e-4))
            with pytest.raises(M.MorayError) as e:
                M.moray_td_step(ctx, td, other)                  # another grid size
            assert e.value.status == M.MORAY_EINVAL
        finally:
            M.moray_td_free(ctx, td)
    finally:
        M.moray_free(ctx)


@pytest.mark.parametrize("precision", [M.MORAY_FP64, M.MORAY_FP32_ACC64])
def test_small_pool_grows_and_matches_a_large_one(precision):
    """A pool of 1024 rays overflows at once and doubles, step after step, as
    the rays in flight grow; every step equals the same step of a state
    created with room for them (counts exactly, fields to summation order)."""
    dev = M.problem_to_device(_problem(4))
    ctx = M.moray_init(device=0, precision=precision)
    big = small = None
    try:
        big = M.moray_td_create(ctx, dev, 4.0, 1 << 21)
        small = M.moray_td_create(ctx, dev, 4.0, 1024)
        for step in range(6):
            want, hw = M.moray_td_step(ctx, big, dev)
            got, hg = M.moray_td_step(ctx, small, dev)
            for k in ("segments", "splits", "rays_escaped", "rays_truncated", "rays_seeded"):
                assert got[k] == want[k], (step, k, got[k], want[k])
            rel, _ = _rel(got["k_ph"][0], _np(want["k_ph"][0]))
            print(f"[td grow p{precision} step {step}] k_ph max rel vs large pool {rel:.2e}, held {hg:.4e}/{hw:.4e}",
                  flush=True)
            assert rel <= 1e-9
            assert hg == pytest.approx(hw, rel=1e-12)
    finally:
        for td in (big, small):
            if td:
                M.moray_td_free(ctx, td)
        M.moray_free(ctx)


def _all_halt(groups, c_dt=4.0):
    """196608 rays of level 7 (none splits) in a thin 16^3 box, all of which halt inside it in the first step."""
    g = W.Grid(np.full((16, 16, 16), 1e-6, np.float32), np.full((16, 16, 16), 0.75, np.float32), W.DX_C1)
    p = W.Problem([g], np.array([[8.1, 7.9, 8.2, 1e49]]), W.hydrogen_spectrum((13.6, 20.0, 30.0, 60.0)[:groups]),
                  W.Params(level_init=7, level_max=7))
    return p, M.problem_to_device(p), c_dt


@pytest.mark.parametrize("precision", [M.MORAY_FP64, M.MORAY_FP32_ACC64])
@pytest.mark.parametrize("groups", [1, 2, 3, 4])
def test_a_pool_holds_as_many_records_as_asked_for(precision, groups):
    """Whatever the groups a record carries. With four waves a compute unit
    every wave of the launch gets an equal share of the 196608 rays, and
    reserves one block of 256 records for them: 262144 in all on 256 compute
    units, the last of which is used up to its 192nd. The context's budget has room
    for 142 bytes a record and what the sort needs besides, but not to grow."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if cus != 256:
        pytest.skip("the records a launch reserves are counted for 256 compute units")
    p, dev, c_dt = _all_halt(groups)
    ref, rays = O.trace_td(p, c_dt, None, emit=True)
    assert len(rays) == 196608 * groups
    pool = 4 * cus * 256
    # 142 B and up to 24 B of sort scratch a record, and 2 MiB of tables
    ctx = M.moray_init(device=0, precision=precision, waves_per_cu=4, hbm_budget_bytes=pool * 166 + (2 << 20))
    td = None
    try:
        td = M.moray_td_create(ctx, dev, c_dt, pool)
        for step in range(2):
            if step:
                ref, rays = O.trace_td(p, c_dt, rays, emit=False)
            res, held = M.moray_td_step(ctx, td, dev, emit=step == 0)
            assert held == pytest.approx(ref["held"], rel=1e-6)
            rel, _ = _rel(res["k_ph"][0], ref["k_ph"][0])
            assert rel <= (1e-9 if precision == M.MORAY_FP64 else 1e-4)
    finally:
        if td:
            M.moray_td_free(ctx, td)
        M.moray_free(ctx)


def test_a_pool_beyond_32_bit_records_is_refused_before_it_is_allocated():
    _, dev, c_dt = _all_halt(1)
    ctx = M.moray_init(device=0, hbm_budget_bytes=1 << 44)
    try:
        free = torch.cuda.mem_get_info()[0]
        with pytest.raises(M.MorayError) as e:
            M.moray_td_create(ctx, dev, c_dt, 1 << 32)
        assert e.value.status == M.MORAY_ENOMEM and "2^32" in str(e.value)
        assert torch.cuda.mem_get_info()[0] == free
    finally:
        M.moray_free(ctx)
