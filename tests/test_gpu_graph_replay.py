"""Captured graphs of the grid kernels against the same kernels launched one
by one (kernel timing), and the sweeps inside them against the oracle, on
systems and shapes that take the grid kernels."""

import numpy as np
import pytest

from paper_2609_21204_amd import dybond as db
from paper_2609_21204_amd import inputs
from test_gpu_parity import assert_in_step_sweep, counters
from test_gpu_resident import assert_same

pytestmark = pytest.mark.gpu


def on_grid(w, shape=(8, 0), **kw):
    s = db.System.from_workload(w, **kw)
    if shape is not None:
        db.db_set_step_shape(s.h, *shape)
    return s


@pytest.mark.parametrize("shape, n, period", [((8, 0), 512, 10), ((2, 0), 512, 7), (None, 1500, 10), (None, 1500, 1)])
def test_graphs_match_single_launches(shape, n, period):
    """Spans (120 steps and more), whole periods, heads, tails and single
    steps; kernel timing launches every kernel by itself."""
    w = inputs.replica(7, n, 3.0, 0.2, 2, "mono")
    w.period = period
    with on_grid(w, shape) as g, on_grid(w, shape) as e:
        db.db_kernel_timing(e.h, 1)
        for steps in (240, 3, 95, 1, 10, 131, 500):
            g.step(steps)
            e.step(steps)
            assert_same(g, e, f"{steps} steps")
        name = "k_step"
        assert db.db_read_kernel_time(e.h, name)[0] == 980 and db.db_read_kernel_time(g.h, name)[0] == 0


def test_sweep_at_the_end_of_a_captured_span_matches_the_oracle():
    w = inputs.small(seed=12)
    with on_grid(w) as s, on_grid(w) as s2:
        s.step(120)
        s2.step(119)
        b0, c0 = s2.bonds().astype(np.int64), counters(s2)
        assert_in_step_sweep(s, w, b0, c0, 120, "span graph, sweep 120")
        s.step(240)
        s2.step(241)
        assert_same(s, s2, "360 steps")


@pytest.mark.parametrize("pre", [29, 5])
def test_sweep_of_one_step_and_one_period_graphs_matches_the_oracle(pre):
    w = inputs.small(seed=6)
    with on_grid(w) as s:
        s.step(pre)
        for rounds in range(3):
            s.step(w.period - 1 - s.step_count % w.period)
            b0, c0 = s.bonds().astype(np.int64), counters(s)
            s.step(1)
            assert_in_step_sweep(s, w, b0, c0, s.step_count, f"sweep {s.step_count}")
            if rounds == 1:
                s.step(w.period)


def test_events_of_a_span_match_those_of_short_calls():
    w = inputs.small(seed=9, eps_bond=2.0)
    with on_grid(w) as g, on_grid(w) as p:
        g.step(240)
        for _ in range(24):
            p.step(10)
        for kind in (db.DB_EVENT_FORMED, db.DB_EVENT_BROKEN):
            eg, sg = g.sweep_events(kind)
            ep, sp = p.sweep_events(kind)
            assert sg == sp == 240 and len(eg) > 0 and np.array_equal(eg, ep)
