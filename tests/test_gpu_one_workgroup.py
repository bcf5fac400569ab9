"""Small systems in one workgroup (state and lists on the chip), through
db_step and db_step_batch, against the grid kernels bit for bit."""

import numpy as np
import pytest

from paper_2609_21204_amd import dybond as db
from paper_2609_21204_amd import inputs
from test_gpu_resident import assert_same

pytestmark = pytest.mark.gpu


def grid_of(w, **kw):
    """The system on the grid kernels (a caller-chosen shape takes them)."""
    s = db.System.from_workload(w, **kw)
    db.db_set_step_shape(s.h, 8, 0)
    return s


def compare(w, calls, what="", **kw):
    """db_step's own choice, a batch and the grid kernels, call by call."""
    with db.System.from_workload(w, **kw) as a, db.System.from_workload(w, **kw) as b, grid_of(w, **kw) as g:
        for steps in calls:
            a.step(steps)
            db.db_step_batch([b.h], steps)
            g.step(steps)
            assert_same(a, g, f"{what} n={w.n}, db_step, {steps} steps")
            assert_same(b, g, f"{what} n={w.n}, batch, {steps} steps")
        return g.observables()


def block(n, rho, spacing, seed=3, kT=1.0, cap=2):
    """n monomers on a cubic lattice in the middle of a box of mean density rho."""
    w = inputs.replica(seed, n, 5.0, rho, cap, "mono", kT=kT)
    m = int(np.ceil(n ** (1.0 / 3.0)))
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
    w.pos = ((g - 0.5 * (m - 1)) * spacing).astype(np.float32)
    return w


@pytest.mark.parametrize("skin", [0.5, 0.8, 1.2])
@pytest.mark.parametrize("n", [130, 384, 400])
def test_lists_that_overflow_on_one_thread_of_a_pair(n, skin):
    """A dense block: with two threads per particle the shares of a list
    differ, and one of them outgrows its 16 LDS slots where the other does
    not (with one thread per particle: 24 slots, some lists longer)."""
    compare(block(n, 0.05, 1.05, kT=0.2), (1, 9, 25), f"skin {skin}", skin=skin)
