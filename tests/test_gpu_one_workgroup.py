"""Small systems in one workgroup (state and lists on the chip), through
db_step and db_step_batch, against the grid kernels bit for bit."""

import math

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


@pytest.mark.parametrize("n, rho", [(300, 0.3), (384, 0.05), (600, 0.3)])
def test_short_calls_build_lists_when_the_grid_kernels_do(n, rho):
    """Both forms build after the same steps and count every build (the one
    of the grid kernels' renumbering at step 0 is before the first count)."""
    w = inputs.replica(9, n, 5.0, rho, 2, "mono")
    with db.System.from_workload(w) as a, grid_of(w) as g:
        a.step(10)
        g.step(10)
        a0, g0 = db.db_read_list_builds(a.h), db.db_read_list_builds(g.h)
        for _ in range(40):
            a.step(5)
            g.step(5)
        assert db.db_read_list_builds(g.h) > g0 + 2
        assert db.db_read_list_builds(a.h) - a0 == db.db_read_list_builds(g.h) - g0
        assert_same(a, g, f"n={n}")


def test_a_call_between_two_builds_meets_no_list_limit():
    """A particle drifts into the list radius of one that already has
    max_neighbors entries, by less than half the skin: no list is built, so
    no call may report that the list is full."""
    w = inputs.Workload(
        name="three", n=3, L=9.0, types=[(0, 1.0, 1.0, 1.0)],
        pos=np.array([[0, 0, 0], [1.2, 0, 0], [-1.44, 0, 0]], np.float32),
        vel=np.array([[0, 0, 0], [0, 0, 0], [1, 0, 0]], np.float32), type_id=np.zeros(3, np.uint32),
        bond_types=[], static_pairs=np.zeros((0, 2), np.uint32), static_types=np.zeros(0, np.uint32),
        reactions=[], kT=1e-9)
    with db.System.from_workload(w, max_neighbors=1) as a, grid_of(w, max_neighbors=1) as g:
        for _ in range(20):
            a.step(1)
            g.step(1)
        assert np.array_equal(a.positions(), g.positions())
        assert -1.42 < a.positions()[2, 0] < -1.3


@pytest.mark.parametrize("n", [300, 700, 1500])
def test_a_sweep_after_every_step_at_the_kinetic_temperature(n):
    """The energy word of the next sweep is cleared while no step adds to it
    (1500 particles: the batch kernel's own loop)."""
    w = inputs.replica(11, n, 3.0, 0.2, 2, "mono")
    w.period = 1
    o = compare(w, (1, 2, 40, 61), "period 1", kt_source=db.DB_KT_KINETIC)
    assert o["forms"].sum() > 0 and o["breaks"].sum() > 0


@pytest.mark.parametrize("n, rho, spacing, grid", [(700, 0.05, 1.13, True), (700, 0.05, 1.8, False), (300, 0.05, 1.13, False),
                                                   (1000, 0.1, 2.0, False), (1000, 0.05, 1.13, True)])
def test_the_form_is_chosen_by_the_lists_not_the_mean_density(n, rho, spacing, grid):
    """A dense block in a large box has long lists: it takes the grid kernels
    (seen by the list build of their renumbering: nothing moves here)."""
    w = block(n, rho, spacing, kT=1e-12)
    w.vel[:] = 0.0
    w.reactions = [dict(w.reactions[0], epsilon=math.nan, k_on=1e-9, k_off=1e-9, p_on0=math.nan)]
    with db.System.from_workload(w) as s:
        b0 = db.db_read_list_builds(s.h)
        s.step(10)
        assert db.db_read_list_builds(s.h) - b0 == (1 if grid else 0)


def test_a_block_that_dissolves_changes_form_within_a_call():
    """Dense at first (grid kernels), dilute later (one workgroup): the same
    trajectory through the changes, with the step counter and the errors of
    one long call."""
    w = block(700, 0.05, 1.05)
    with db.System.from_workload(w) as a, grid_of(w) as g:
        for steps in (3, 6000, 2500, 17):
            a.step(steps)
            g.step(steps)
            assert a.step_count == g.step_count
            assert_same(a, g, f"{steps} steps")


def three_reactions(seed, n):
    """Telechelic chains whose ends (valence 2) bind crosslinkers and, not
    within their own molecule, each other; crosslinkers bind each other too."""
    w = inputs.replica(seed, n, 4.0, 0.3, 4, "chains")
    w.types[0] = (2,) + tuple(w.types[0][1:])
    w.bond_types = list(w.bond_types) + [(inputs.HARMONIC, 80.0, 1.0), (inputs.HARMONIC, 60.0, 1.05)]
    r = w.reactions[0]
    w.reactions = [dict(r, epsilon=2.0), dict(r, type_a=0, type_b=0, bond_type=2, epsilon=1.5, p_on0=0.8, self_avoid=1),
                   dict(r, type_a=2, type_b=2, bond_type=3, epsilon=1.0, p_on0=0.5)]
    return w


@pytest.mark.parametrize("n", [300, 600])
def test_several_reactions_in_one_sweep(n):
    o = compare(three_reactions(21, n), (9, 1, 60, 130), "three reactions")
    assert (o["forms"] > 0).all() and (o["breaks"] > 0).all(), o


@pytest.mark.parametrize("n", [300, 600])
def test_more_bond_slots_than_words_in_registers(n):
    o = compare(inputs.gel_lattice(seed=4, n=n, eps_ab=3.0, eps_ac=2.0), (50, 3, 150), "gel", kt_source=db.DB_KT_KINETIC)
    assert (o["forms"] > 0).all() and (o["breaks"] > 0).all(), o


@pytest.mark.parametrize("n", [200, 384, 500])
@pytest.mark.parametrize("kind", ["slip", "slip+tether", "melt+kinetic"])
def test_full_variant(kind, n):
    """Rate modifiers and tether bonds with one and two threads per particle."""
    w = inputs.replica(13, n, 3.0, 0.25, 2, "mono")
    r, kt = w.reactions[0], db.DB_KT_SETPOINT
    if "slip" in kind:
        r["slip"] = 0.5
    if "tether" in kind:
        w.bond_types = [(db.DB_BOND_TETHER, 2.0, 0.5, 0.8, 1.2, 1.6)]
        r.update(r_min=0.6, r_max=1.5)
    if "melt" in kind:
        from test_gpu_modifiers import _melt_half_bound
        r.update(epsilon=5.0, melt=_melt_half_bound())
        kt = db.DB_KT_KINETIC
    o = compare(w, (31, 9, 160), kind, kt_source=kt)
    assert o["forms"].sum() > 0 and o["breaks"].sum() > 0


@pytest.mark.parametrize("n, rho, skin", [(30, 0.4, None), (31, 0.4, None), (46, 0.45, None), (49, 0.4, 0.9), (50, 0.4, 0.9),
                                          (99, 0.4, 0.9), (114, 0.45, 0.9)])
def test_boxes_of_three_cells(n, rho, skin):
    """Boxes that shrink the skin to what three cells leave it, in which L
    over the cell side rounds to just below 3."""
    w = inputs.replica(2, n, 4.0, rho, 2, "mono")
    room = w.L / (3.0 * (1.0 + 1e-5)) - 1.3
    assert 0.0 < room and w.L / ((1.3 + min(0.3 if skin is None else skin, room)) * (1.0 + 1e-5)) < 3.0
    compare(w, (1, 20, 60), f"skin {skin}", skin=skin)
