"""The step kernel that deals its force work out through queues (2 and 4
threads per particle) against the one with a particle's work on its own
threads (8), bit for bit: workgroups that are not full, queues that overflow,
every kind of bond, and the kinetic temperature."""

import numpy as np
import pytest

from paper_2609_21204_amd import dybond as db
from paper_2609_21204_amd import inputs
from test_gpu_resident import assert_same

pytestmark = pytest.mark.gpu
SHAPES = [(2, 0), (4, 1), (4, 2), (4, 4), (1, 0)]


def compare(w, shape, calls, **kw):
    with db.System.from_workload(w, **kw) as a, db.System.from_workload(w, **kw) as b:
        db.db_set_step_shape(a.h, *shape)
        db.db_set_step_shape(b.h, 8, 0)
        for steps in calls:
            a.step(steps)
            b.step(steps)
            assert_same(a, b, f"n={w.n}, shape {shape}, {steps} steps")


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("n, kind", [(127, "mono"), (129, "mono"), (2050, "chains")])
def test_workgroups_that_are_not_full(n, kind, shape):
    compare(inputs.replica(17, n, 7.0, 0.3, 4, kind), shape, (1, 60, 80), kt_source=db.DB_KT_KINETIC)


@pytest.mark.parametrize("shape", SHAPES)
def test_more_pairs_than_the_queue_holds(shape):
    """60 and more listed neighbours per particle (no WCA), and a small dense
    box in which a third of the pairs cross the boundary and take the FP64
    evaluation: both queues overflow."""
    w = inputs.replica(5, 600, 4.0, 0.2, 2, "mono")
    rng = np.random.default_rng(3)
    w.types = [(v, 0.0, 1.0, 1.0) for v, _, _, _ in w.types]
    w.pos = (w.pos * 0.1 + rng.normal(0, 0.25, w.pos.shape)).astype(np.float32)
    w.kT = 0.05
    compare(w, shape, (5, 40), max_neighbors=1024)
    compare(inputs.replica(6, 100, 5.0, 0.85, 2, "mono"), shape, (25, 40))


@pytest.mark.parametrize("shape", SHAPES)
def test_full_variant_with_many_bond_slots(shape):
    """Six-valent sites with slip bonds beside a tether bond type."""
    w = inputs.gel_lattice(seed=4, n=3000)
    w.bond_types = list(w.bond_types) + [(db.DB_BOND_TETHER, 2.0, 0.5, 0.8, 1.2, 1.6)]
    for r in w.reactions:
        r["slip"] = 0.5
    compare(w, shape, (150, 90))


@pytest.mark.parametrize("shape, batch", [((1, 0), 4), ((2, 0), 3), ((2, 4), 3), ((4, 0), 1), ((4, 2), 2), ((4, 4), 4),
                                          ((8, 0), 1), ((16, 0), 1), ((32, 0), 1)])
def test_the_shape_in_use_is_the_one_that_is_launched(shape, batch):
    with db.System.from_workload(inputs.replica(3, 200, 5.0, 0.2, 2, "mono"), commit=False) as s:
        db.db_set_step_shape(s.h, *shape)
        assert db.db_get_step_shape(s.h) == shape                # as requested
        db.db_commit(s.h)
        assert db.db_get_step_shape(s.h) == (shape[0], batch)    # as resolved
