"""The bonds of a sweep's list against the bond tables before and after it, at
the sizes where the claim kernel's workgroups (which append to that list
together) end ragged or become wider."""

import numpy as np
import pytest

from paper_2609_21204_amd import dybond as db
from paper_2609_21204_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1025, 33000, (1 << 19) - 1, 1 << 19, (1 << 19) + 1])
def test_event_lists_are_the_change_of_the_bonds(n):
    def rows(t):
        t = np.asarray(t).astype(np.uint64)
        return (t[:, 0] << np.uint64(32)) | (t[:, 1] << np.uint64(8)) | t[:, 2]

    w = inputs.gel_lattice(seed=3, n=n)
    with db.System.from_workload(w) as s:
        db.db_set_step_shape(s.h, 8 if n < 32768 else 2, 0)     # grid kernels at every size
        s.step(2 * w.period - 1)
        before = rows(s.bonds())
        s.step(1)
        after = rows(s.bonds())
        (formed, key), (broken, _) = s.sweep_events(db.DB_EVENT_FORMED), s.sweep_events(db.DB_EVENT_BROKEN)
        o = s.observables()
    assert key == 2 * w.period and len(formed) > n // 2000
    formed, broken = rows(formed), rows(broken)
    assert len(np.unique(formed)) == len(formed)
    assert np.array_equal(np.sort(np.concatenate([before, formed])), np.sort(np.concatenate([after, broken])))
    assert int(o["forms"].sum()) - int(o["breaks"].sum()) == len(after)
