"""Rays that carry several energy groups, and the launch rules beside them, against
the oracle at the sizes where they can go wrong.

Bars: those of checks.check (per cell 1e-9 in float64 and 1e-4 in mixed precision
where the oracle exceeds 1e-6 of its maximum; ledger exact), derived there.
"""
import numpy as np
import pytest

from checks import check as _check
from oracle import oracle as O
from paper_1012_2865_amd import moray as M
from paper_1012_2865_amd import workloads as W

pytestmark = pytest.mark.gpu

ENERGIES = (13.6, 20.0, 30.0, 60.0, 40.0, 17.0)
PRECISIONS = {"fp64": M.MORAY_FP64, "fp32": M.MORAY_FP32_ACC64}
BAR = {"fp64": 1e-9, "fp32": 1e-4}


def _box(item, sides, groups, sources=2, mean=1e-2, params=None):
    """A lognormal box of unequal sides: neutral and dense enough for the softer groups to end in it."""
    rng = W.rng_for(97, item, 0)
    nx, ny, nz = sides
    n_h = (mean * np.exp(rng.normal(0.0, 1.0, (nz, ny, nx)))).astype(np.float32)
    x_hi = rng.uniform(0.5, 1.0, (nz, ny, nx)).astype(np.float32)
    pos = rng.uniform(0.0, 1.0, (sources, 3)) * (np.array(sides) - 1e-6)
    src = np.column_stack([pos, 10.0 ** rng.uniform(48.0, 50.0, sources)])
    return W.Problem([W.Grid(n_h, x_hi, 64.0 * W.DX_C1)], src, W.hydrogen_spectrum(ENERGIES[:groups]),
                     params or W.Params())


def _held(name, problems, context=None, **init):
    """Each problem of one batched call against the oracle."""
    ctx = M.moray_init(precision=PRECISIONS[name], **init)
    try:
        res = M.moray_trace(ctx, [M.problem_to_device(p) for p in problems])
        for k, p in enumerate(problems):
            _check(res[k], O.trace(p), BAR[name], name=f"{name} {context} {k}", fp64=name == "fp64")
    finally:
        M.moray_free(ctx)


@pytest.mark.parametrize("name", list(PRECISIONS))
@pytest.mark.parametrize("groups", [1, 2, 3, 4, 5, 6])
def test_groups_per_ray(name, groups):
    # one pack, a full one, and a second of one and two; groups that end on the way
    _held(name, [_box(1, (21, 17, 19), groups)], groups)


@pytest.mark.parametrize("name", list(PRECISIONS))
def test_batch_of_unlike_groups_and_odd_cells(name):
    # one and several sums a cell side by side, their first cells anywhere in a line
    _held(name, [_box(2, (9, 7, 5), 1), _box(3, (13, 11, 3), 4), _box(4, (7, 17, 9), 1), _box(5, (5, 5, 5), 6)],
          "mixed batch")


@pytest.mark.parametrize("name", list(PRECISIONS))
@pytest.mark.parametrize("level_init,level_max,phi_c", [(0, 3, 5.1), (2, 12, 5.1), (4, 4, 5.1), (3, 5, 2.1), (1, 12, 9.0)])
def test_seeds_at_a_finer_level(name, level_init, level_max, phi_c):
    params = W.Params(level_init=level_init, level_max=level_max, phi_c=phi_c)
    _held(name, [_box(6, (23, 18, 20), 3, params=params)], (level_init, level_max, phi_c))


@pytest.mark.parametrize("name", list(PRECISIONS))
def test_batch_of_unlike_first_levels(name):
    # seeds of unlike levels enter at their own
    _held(name, [_box(7, (11, 12, 13), 2, params=W.Params(level_init=k)) for k in (0, 2, 3)], "first levels")


@pytest.mark.parametrize("chunk_rays", [1, 64, 100, 4096])
def test_units_of_any_size(chunk_rays):
    # more rays than one unit for every wave of one block a CU, dealt and claimed
    _held("fp32", [_box(8, (64, 61, 58), 4, sources=12, mean=1e-5)], chunk_rays, chunk_rays=chunk_rays, waves_per_cu=4)


@pytest.mark.parametrize("name", list(PRECISIONS))
def test_rays_longer_than_a_frame(name):
    # axis-parallel rays that never split cross 4090 cells: past the 2048 steps after
    # which mixed precision forms its plane distances afresh
    p = _box(9, (4096, 3, 2), 2, sources=1, mean=1e-6, params=W.Params(level_init=0, level_max=0))
    p.sources[0, :3] = (2.5, 1.5, 0.75)
    _held(name, [p], "long")


@pytest.mark.parametrize("name", list(PRECISIONS))
def test_serving_of_unlike_groups_and_odd_cells(name):
    probs = [_box(10, (9, 7, 5), 1), _box(11, (11, 9, 7), 3), _box(12, (5, 7, 3), 1), _box(13, (13, 9, 11), 6)]
    ctx = M.moray_init(precision=PRECISIONS[name])
    try:
        tickets = [M.moray_trace_async(ctx, [M.problem_to_device(p)]) for p in probs]
        for k, (t, p) in enumerate(zip(tickets, probs)):
            _check(M.moray_query(ctx, t)[0], O.trace(p), BAR[name], name=f"{name} serving {k}", fp64=name == "fp64")
    finally:
        M.moray_free(ctx)


def test_thin_marks_of_odd_counts():
    # marks cleared 16 at a time and read 8 at a time: neither divides 9 trees of 693 cells
    p = _box(14, (11, 9, 7), 3, sources=3, mean=1e-5, params=W.Params(tau_thin=0.1))
    ref = O.trace(p)
    ctx = M.moray_init(precision=M.MORAY_FP64)
    try:
        for _ in range(2):                        # the second pass finds the first one's marks
            res = M.moray_trace(ctx, [M.problem_to_device(p)])[0]
            for f in ("k_ph", "heating"):
                np.testing.assert_allclose(np.asarray(res[f][0].cpu()).ravel(), np.asarray(ref[f][0]).ravel(), rtol=1e-9)
    finally:
        M.moray_free(ctx)


def _finite(res, name):
    for f in ("k_ph", "heating"):
        for q, v in enumerate(res[f]):
            assert bool(np.isfinite(np.asarray(v.cpu())).all()), (name, f, q)


@pytest.mark.parametrize("name", list(PRECISIONS))
@pytest.mark.parametrize("narrow", [1, 2])
def test_serving_rays_get_wider(monkeypatch, name, narrow):
    # A request of one or two groups runs alone for a launch; then one of four joins (its own
    # seed level keeps the two from entering together), and the launch reads four rates of rays
    # that were queued with fewer. What the queue held there before must not matter: NaN here.
    # Units of one ray put narrow and wide rays into the same waves.
    first = _box(15, (48, 45, 47), narrow, sources=3, mean=1e-5, params=W.Params(level_init=1))
    then = _box(16, (40, 44, 41), 4, sources=2, mean=1e-5, params=W.Params(level_init=2))
    monkeypatch.setenv("MORAY_INJECT_SERVE_STALE_RATES", "1")
    ctx = M.moray_init(precision=PRECISIONS[name], chunk_rays=1, waves_per_cu=4, queue_capacity=1 << 24)
    monkeypatch.delenv("MORAY_INJECT_SERVE_STALE_RATES")
    try:
        tickets = [M.moray_trace_async(ctx, [M.problem_to_device(p)]) for p in (first, then)]
        res = [M.moray_query(ctx, t)[0] for t in tickets]
        assert res[0]["t_admit"] < res[1]["t_admit"] < res[0]["t_done"]       # it did join a running launch sequence
        for r, p, k in zip(res, (first, then), ("narrow", "wide")):
            _finite(r, k)
            _check(r, O.trace(p), BAR[name], name=f"{name} {k}", fp64=name == "fp64")
    finally:
        M.moray_free(ctx)


def _nested_box(item, groups, **params):
    """A box with a 2x-refined child that holds one of the sources; two packs from five groups on."""
    p = _box(item, (20, 17, 18), groups, sources=3, mean=3e-3, params=W.Params(**params))
    rng = W.rng_for(97, 100 + item, 0)
    child = W.Grid((3e-3 * np.exp(rng.normal(0.0, 1.0, (8, 12, 10)))).astype(np.float32),
                   rng.uniform(0.5, 1.0, (8, 12, 10)).astype(np.float32), p.grids[0].dx_cm / 2, parent=0, offset=(7, 4, 6))
    p.grids.append(child)
    p.sources[0, :3] = (9.3, 7.1, 8.2)
    return p


@pytest.mark.parametrize("name", list(PRECISIONS))
@pytest.mark.parametrize("groups", [2, 5, 6])
def test_packs_cross_nested_grids(name, groups):
    _held(name, [_nested_box(17, groups)], groups)


@pytest.mark.parametrize("name", list(PRECISIONS))
@pytest.mark.parametrize("groups", [3, 5, 6])
def test_packs_with_the_covering_factor(name, groups):
    p = _nested_box(18, groups, covering=True)
    ctx = M.moray_init(precision=PRECISIONS[name])
    try:
        res = M.moray_trace(ctx, [M.problem_to_device(p)])[0]
    finally:
        M.moray_free(ctx)
    _check(res, O.trace(p), BAR[name], name=f"{name} covering {groups}", fp64=name == "fp64", conserving=False)


@pytest.mark.parametrize("name", list(PRECISIONS))
@pytest.mark.parametrize("groups", [5, 6])
def test_packs_of_time_dependent_rays(name, groups):
    # groups that end in different steps, rays that halt and are taken up again, splits on the way
    p = _nested_box(19, groups)
    dev, c_dt = M.problem_to_device(p), 5.0
    ctx = M.moray_init(precision=PRECISIONS[name])
    td = None
    try:
        td = M.moray_td_create(ctx, dev, c_dt, 1 << 20)
        rays = None
        for step, emit in enumerate([True, True, False, True]):
            ref, rays = O.trace_td(p, c_dt, rays, emit=emit)
            res, held = M.moray_td_step(ctx, td, dev, emit=emit)
            for q in range(2):
                want = np.asarray(ref["k_ph"][q]).ravel()
                got = np.asarray(res["k_ph"][q].cpu()).ravel()
                m = want > 1e-6 * want.max()
                assert np.max(np.abs(got[m] / want[m] - 1.0)) <= BAR[name], (step, q)
            assert held == pytest.approx(ref["held"], rel=BAR[name])
            if name == "fp64":
                for k in ("segments", "splits", "rays_escaped", "rays_truncated"):
                    assert res[k] == ref["totals"][k], (step, k)
    finally:
        if td:
            M.moray_td_free(ctx, td)
        M.moray_free(ctx)


@pytest.mark.parametrize("name", list(PRECISIONS))
def test_one_option_in_a_batch_of_packs(name):
    # an optically-thin problem puts every ray of its batch back to one group: same results
    probs = [_box(20, (13, 9, 11), 4), _box(21, (11, 12, 9), 4, mean=1e-5, params=W.Params(tau_thin=0.05)), _nested_box(22, 5)]
    ctx = M.moray_init(precision=PRECISIONS[name])
    try:
        res = M.moray_trace(ctx, [M.problem_to_device(p) for p in probs])
    finally:
        M.moray_free(ctx)
    for k in (0, 2):
        _check(res[k], O.trace(probs[k]), BAR[name], name=f"{name} beside a thin problem {k}", fp64=name == "fp64")


@pytest.mark.parametrize("name", list(PRECISIONS))
@pytest.mark.parametrize("groups", [1, 2, 4, 6])
def test_packs_without_the_deposit_cache(name, groups):
    _held(name, [_nested_box(23, groups), _box(24, (9, 7, 5), 1), _box(25, (13, 11, 3), groups)], groups, deposit_cache=-1)


@pytest.mark.parametrize("name", list(PRECISIONS))
def test_radiation_pressure_without_the_deposit_cache(name):
    p = _nested_box(26, 3)
    dev = M.problem_to_device(p)
    res = []
    for cache in (0, -1):
        ctx = M.moray_init(precision=PRECISIONS[name], deposit_cache=cache)
        try:
            res.append(M.moray_trace(ctx, [dev], want_accel=True)[0])
        finally:
            M.moray_free(ctx)
        _check(res[-1], O.trace(p), BAR[name], name=f"{name} cache {cache}", fp64=name == "fp64")
    # the same segments, added in another order
    for q in range(2):
        a, b = (np.asarray(r["accel"][q].cpu()) for r in res)
        assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))
