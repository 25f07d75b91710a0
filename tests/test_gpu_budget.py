"""The HBM budget of a context across its calls: the ray queue gets what the
other buffers leave, counting the context's own buffers of earlier calls as
what they are, its to use again."""
import numpy as np
import pytest
import torch

from paper_1012_2865_amd import moray as M
from paper_1012_2865_amd import workloads as W

pytestmark = pytest.mark.gpu

COUNTS = ("segments", "splits", "rays_seeded", "rays_escaped", "rays_truncated")


def _same(got, want):
    for k in COUNTS:
        assert got[k] == want[k], (k, got[k], want[k])
    a, b = (r["k_ph"][0].cpu().numpy().ravel() for r in (got, want))
    assert np.allclose(a, b, rtol=1e-9, atol=1e-9 * b.max())


@pytest.mark.parametrize("out_on_device", [True, False])
def test_a_queue_that_fills_the_budget_serves_later_calls(out_on_device):
    # eight trees of up to 1.4 million rays a level; room for about 2.5 million rays after the
    # other buffers and the 64 MiB the planner leaves
    p = M.problem_to_device(W.lognormal_problem(97, 60, 96, 8))
    small = M.problem_to_device(W.lognormal_problem(97, 61, 24, 2))
    free = M.moray_init(device=0)
    tight = M.moray_init(device=0, hbm_budget_bytes=190 << 20)
    try:
        want, want_small = (M.moray_trace(free, [q])[0] for q in (p, small))
        for call in range(3):
            kw = {} if out_on_device else {"out_on_device": False}
            got = M.moray_trace(tight, [p], **kw)[0]
            print(f"call {call}: peak {got['peak_level_rays']}, launches {got['trace_launches']}", flush=True)
            if not out_on_device:
                got = dict(got, k_ph=[torch.as_tensor(np.asarray(a)) for a in got["k_ph"]])
            _same(got, want)
            _same(M.moray_trace(tight, [small])[0], want_small)
    finally:
        M.moray_free(free)
        M.moray_free(tight)


def test_other_states_of_a_context_are_not_the_queues():
    # a pool of time-dependent rays takes most of the budget: the trace beside it gets the rest
    p = M.problem_to_device(W.lognormal_problem(97, 60, 96, 8))
    free = M.moray_init(device=0)
    ctx = M.moray_init(device=0, hbm_budget_bytes=700 << 20)
    td = None
    try:
        want = M.moray_trace(free, [p])[0]
        td = M.moray_td_create(ctx, p, 24.0, 3 << 20)
        for _ in range(2):
            _same(M.moray_trace(ctx, [p])[0], want)
    finally:
        if td:
            M.moray_td_free(ctx, td)
        M.moray_free(free)
        M.moray_free(ctx)


def test_a_queue_of_wide_rays_after_one_of_narrow_rays():
    # the same budget filled with slots of one rate, then of four, then of one
    many = M.problem_to_device(W.lognormal_problem(97, 60, 96, 8))
    one = M.problem_to_device(W.lognormal_problem(97, 60, 96, 8, energies=(13.6,)))
    free = M.moray_init(device=0)
    tight = M.moray_init(device=0, hbm_budget_bytes=190 << 20)
    try:
        for p in (one, many, one, many):
            _same(M.moray_trace(tight, [p])[0], M.moray_trace(free, [p])[0])
    finally:
        M.moray_free(free)
        M.moray_free(tight)
