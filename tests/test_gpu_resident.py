"""One-workgroup runs with the state on the chip against the grid kernels, bit
for bit, at the edges of their layouts: one and two threads per particle (384
particles), whole and partial waves, the largest size (1024), lists that
overflow their LDS slots, and the errors both paths report."""

import numpy as np
import pytest

from paper_2609_21204_amd import dybond as db
from paper_2609_21204_amd import inputs

pytestmark = pytest.mark.gpu


def state(s):
    pos, img = s.positions(with_images=True)
    ev = [s.sweep_events(w)[0] for w in (db.DB_EVENT_FORMED, db.DB_EVENT_BROKEN)]
    o = s.observables()
    return [pos, img, s.velocities(), s.forces(), s.bonds(), *ev, o["attempts"], o["forms"], o["breaks"]]


def assert_same(a, b, what):
    for k, (x, y) in enumerate(zip(state(a), state(b))):
        assert np.array_equal(x, y), f"{what}: item {k}"


@pytest.mark.parametrize("n, rho, kind", [(40, 0.05, "mono"), (63, 0.3, "mono"), (64, 0.3, "mono"), (65, 0.2, "chains"),
                                          (384, 0.3, "mono"), (385, 0.3, "mono"), (700, 0.35, "chains"),
                                          (1023, 0.05, "mono"), (1024, 0.4, "mono"), (1025, 0.1, "mono")])
def test_batched_runs_match_the_grid_kernels(n, rho, kind):
    w = inputs.replica(31, n, 6.0, rho, 2, kind)
    with db.System.from_workload(w) as a, db.System.from_workload(w) as b:
        db.db_set_step_shape(b.h, 8, 0)            # a caller-chosen shape takes the grid kernels
        for steps in (7, 1, 53, 130):
            db.db_step_batch([a.h], steps)
            b.step(steps)
            assert_same(a, b, f"{steps} steps")
        a.step(33)                                  # db_step's own choice
        b.step(33)
        assert_same(a, b, "after db_step")


def test_lists_longer_than_their_lds_slots():
    """sigma 0 switches WCA off, so particles may sit on top of each other: 60
    neighbours per particle, more than the 24 (or 2 x 16) LDS slots."""
    for n in (200, 600):
        w = inputs.replica(5, n, 4.0, 0.2, 2, "mono")
        rng = np.random.default_rng(3)
        w.types = [(v, 0.0, 1.0, 1.0) for v, _, _, _ in w.types]
        w.pos = (w.pos * (0.05 if n == 200 else 0.1) + rng.normal(0, 0.25, w.pos.shape)).astype(np.float32)
        w.kT = 0.05
        with db.System.from_workload(w, max_neighbors=1024) as a, db.System.from_workload(w, max_neighbors=1024) as b:
            db.db_set_step_shape(b.h, 8, 0)
            for steps in (5, 40, 41):
                db.db_step_batch([a.h], steps)
                b.step(steps)
                assert_same(a, b, f"n={n}, {steps} steps")


def test_a_list_beyond_max_neighbors_is_an_error():
    w = inputs.replica(5, 300, 4.0, 0.35, 2, "mono")
    with db.System.from_workload(w, max_neighbors=30) as s:
        pos = (w.pos * 0.99).astype(np.float32)
        vel = (w.vel + np.where(w.pos > 0, -60.0, 60.0)).astype(np.float32)      # implode: lists outgrow 30 entries
        s.set_state(0, pos, vel)
        with pytest.raises(db.DybondError) as e:
            for _ in range(20):
                db.db_step_batch([s.h], 5)
        assert e.value.name in ("DB_EOVERFLOW", "DB_EBOND")
        with pytest.raises(db.DybondError) as e:
            s.step(1)
        assert e.value.name == "DB_ESTATE"
