"""ctypes binding of the C ABI in include/dybond.h (argument marshalling only).

Every function named ``db_*`` here calls the C function of the same name in
``libdybond.so``; arrays are passed as contiguous numpy buffers and a
non-OK status raises :class:`DybondError`.  All computation happens in the
HIP library; if the library has not been built this module raises instead of
falling back to anything else.
"""

import ctypes
import math
import os

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libdybond.so")

DB_OK, DB_EINVAL, DB_ENOMEM, DB_EDEVICE, DB_ESTATE, DB_ERANGE, DB_EBOND, DB_ETRUNC, DB_EOVERFLOW = range(9)
STATUS_NAMES = ["DB_OK", "DB_EINVAL", "DB_ENOMEM", "DB_EDEVICE", "DB_ESTATE", "DB_ERANGE",
                "DB_EBOND", "DB_ETRUNC", "DB_EOVERFLOW"]
DB_BOND_HARMONIC, DB_BOND_FENE, DB_BOND_TETHER = 0, 1, 2
DB_KT_SETPOINT, DB_KT_KINETIC = 0, 1
DB_EVENT_FORMED, DB_EVENT_BROKEN = 0, 1
NO_SWEEP = 2 ** 64 - 1
MAX_RX = 8


class DybondError(RuntimeError):
    def __init__(self, status, message):
        name = STATUS_NAMES[status] if 0 <= status < len(STATUS_NAMES) else str(status)
        super().__init__(f"{name}: {message}")
        self.status = status
        self.name = name


class ReactionDesc(ctypes.Structure):
    _fields_ = [("type_a", ctypes.c_uint32), ("type_b", ctypes.c_uint32),
                ("bond_type", ctypes.c_uint32),
                ("r_min", ctypes.c_double), ("r_max", ctypes.c_double),
                ("k_on", ctypes.c_double), ("k_off", ctypes.c_double),
                ("epsilon", ctypes.c_double), ("p_on0", ctypes.c_double),
                ("self_avoid", ctypes.c_int32)]


class Observables(ctypes.Structure):
    _fields_ = [("step", ctypes.c_uint64), ("n_reactions", ctypes.c_uint32),
                ("pad", ctypes.c_uint32),
                ("n_bonds", ctypes.c_uint64 * MAX_RX), ("attempts", ctypes.c_uint64 * MAX_RX),
                ("forms", ctypes.c_uint64 * MAX_RX), ("breaks", ctypes.c_uint64 * MAX_RX),
                ("bonded_fraction", ctypes.c_double * MAX_RX),
                ("largest_cluster_fraction", ctypes.c_double),
                ("pe", ctypes.c_double), ("ke", ctypes.c_double), ("t_kin", ctypes.c_double)]


_P = ctypes.c_void_p
_U32 = ctypes.c_uint32
_U64 = ctypes.c_uint64
_D = ctypes.c_double
_I = ctypes.c_int
BATCH_MAX_CLASSES = 8


class BatchPlan(ctypes.Structure):
    _fields_ = [("n_classes", ctypes.c_uint32), ("n_max", ctypes.c_uint32 * BATCH_MAX_CLASSES),
                ("threads", ctypes.c_uint32 * BATCH_MAX_CLASSES)]


_SIGS = {
    "db_create": (_I, [_U32, _U32, _D, _U32, _I, ctypes.POINTER(_P)]),
    "db_destroy": (None, [_P]),
    "db_set_type": (_I, [_P, _U32, _U32, _D, _D, _D]),
    "db_set_particles": (_I, [_P, _P, _P, _P]),
    "db_add_bond_type": (_I, [_P, _I, _D, _D, ctypes.POINTER(_U32)]),
    "db_add_tether_bond_type": (_I, [_P, _D, _D, _D, _D, _D, ctypes.POINTER(_U32)]),
    "db_set_reaction_melting": (_I, [_P, _U32, _D, _D, _D, _D]),
    "db_set_reaction_slip": (_I, [_P, _U32, _D]),
    "db_set_temperature": (_I, [_P, _D]),
    "db_add_static_bonds": (_I, [_P, _P, _P, _U64]),
    "db_add_reaction": (_I, [_P, ctypes.POINTER(ReactionDesc), ctypes.POINTER(_U32)]),
    "db_set_integrator": (_I, [_P, _D, _D, _D, _U32, _I]),
    "db_set_cell_capacity": (_I, [_P, _U32]),
    "db_set_neighbor_list": (_I, [_P, _D, _U32]),
    "db_set_matching": (_I, [_P, _U32, _U32]),
    "db_set_step_shape": (_I, [_P, _U32, _U32]),
    "db_get_step_shape": (_I, [_P, ctypes.POINTER(_U32), ctypes.POINTER(_U32)]),
    "db_validate": (_I, [_P]),
    "db_get_reaction": (_I, [_P, _U32, ctypes.POINTER(ReactionDesc), ctypes.POINTER(_D), ctypes.POINTER(_D)]),
    "db_commit": (_I, [_P]),
    "db_step": (_I, [_P, _U64]),
    "db_step_batch": (_I, [_P, _U32, _U64]),
    "db_step_batch_plan": (_I, [_P, _U32, _U64, ctypes.POINTER(BatchPlan)]),
    "db_set_batch_plan": (_I, [_I, ctypes.POINTER(BatchPlan)]),
    "db_get_batch_plan": (_I, [_I, ctypes.POINTER(BatchPlan)]),
    "db_batch_autotune": (_I, [_P, _U32, _U32, ctypes.POINTER(BatchPlan), ctypes.POINTER(_U64), _P, _U32]),
    "db_sweep_frozen": (_I, [_P, _U64]),
    "db_set_state": (_I, [_P, _U64, _P, _P, _P, _P, _U64]),
    "db_save_checkpoint": (_I, [_P, _P, _U64, ctypes.POINTER(_U64)]),
    "db_load_checkpoint": (_I, [_P, _P, _U64]),
    "db_read_positions": (_I, [_P, _P, _P]),
    "db_read_velocities": (_I, [_P, _P]),
    "db_read_forces": (_I, [_P, _P]),
    "db_read_bonds": (_I, [_P, _P, _P, _U64, ctypes.POINTER(_U64)]),
    "db_read_bonds_noalloc": (_I, [_P, _P, _P, _U64, ctypes.POINTER(_U64)]),
    "db_read_sweep_events": (_I, [_P, ctypes.c_int, _P, _P, _U64, ctypes.POINTER(_U64), ctypes.POINTER(_U64)]),
    "db_read_observables": (_I, [_P, ctypes.POINTER(Observables)]),
    "db_bond_reference": (_I, [_P]),
    "db_bond_correlation": (_I, [_P, ctypes.POINTER(_U64), ctypes.POINTER(_U64)]),
    "db_bond_multiplicity": (_I, [_P, _P, _U32, ctypes.POINTER(_U64), ctypes.POINTER(_U64)]),
    "db_cluster_sizes": (_I, [_P, _P, _U32, ctypes.POINTER(_U64)]),
    "db_read_positions_device": (_I, [_P, _P, _P]),
    "db_read_velocities_device": (_I, [_P, _P, _P]),
    "db_read_forces_device": (_I, [_P, _P, _P]),
    "db_get_step": (_U64, [_P]),
    "db_read_list_builds": (_I, [_P, ctypes.POINTER(_U64)]),
    "db_last_error": (ctypes.c_char_p, [_P]),
    "db_set_stream": (_I, [_P, _P]),
    "db_kernel_timing": (_I, [_P, _I]),
    "db_read_kernel_time": (_I, [_P, ctypes.c_char_p, ctypes.POINTER(_U64), ctypes.POINTER(_D)]),
    # surrogate network (include/dybond_mlp.h)
    "db_mlp_create": (_I, [_U32, _I, ctypes.POINTER(_P)]),
    "db_mlp_destroy": (None, [_P]),
    "db_mlp_set_params": (_I, [_P, _P, _U64]),
    "db_mlp_get_params": (_I, [_P, _P, _U64]),
    "db_mlp_predict": (_I, [_P, _P, _U64, _P]),
    "db_mlp_loss_grad": (_I, [_P, _P, _P, _U32, ctypes.POINTER(ctypes.c_float), _P]),
    "db_mlp_train": (_I, [_P, _P, _P, _U64, _U32, _U32, ctypes.c_float, _U64, ctypes.POINTER(ctypes.c_float)]),
    "db_mlp_last_error": (ctypes.c_char_p, [_P]),
}

MLP_PARAMS = 17410

_lib = None


def load():
    """Load libdybond.so (raises if it has not been built)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: build it with __graft_entry__.build()")
        # PyTorch for ROCm carries its own HIP runtime under the soname the
        # library links against; loaded first, it is the one the library
        # binds to, so that the process holds a single runtime (a second
        # copy loaded after the library's would find no device)
        try:
            import torch  # noqa: F401
        except ImportError:
            pass
        lib = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in _SIGS.items():
            fn = getattr(lib, name)
            fn.restype = res
            fn.argtypes = args
        _lib = lib
    return _lib


def _check(handle, status):
    if status != DB_OK:
        msg = load().db_last_error(handle)
        raise DybondError(status, msg.decode() if msg else "")


def _buf(a, dtype):
    a = np.ascontiguousarray(a, dtype=dtype)
    return a, a.ctypes.data_as(_P)


# ---------------------------------------------------------------- thin wrappers
def db_create(n, n_types, box_L, seed, device=0):
    h = _P()
    st = load().db_create(n, n_types, box_L, seed, device, ctypes.byref(h))
    _check(None, st)
    return h


def db_destroy(h):
    load().db_destroy(h)


def db_set_type(h, t, valence, sigma, eps, mass):
    _check(h, load().db_set_type(h, t, valence, sigma, eps, mass))


def db_set_particles(h, pos, vel, types):
    """vel=None: Maxwell-Boltzmann velocities drawn by the library."""
    p, pp = _buf(pos, np.float32)
    v, vp = (None, None) if vel is None else _buf(vel, np.float32)
    t, tp = _buf(types, np.uint32)
    _check(h, load().db_set_particles(h, pp, vp, tp))


def db_add_bond_type(h, kind, k, r0):
    i = _U32()
    _check(h, load().db_add_bond_type(h, kind, k, r0, ctypes.byref(i)))
    return i.value


def db_add_tether_bond_type(h, k_b, l_min, l_c1, l_c0, l_max):
    i = _U32()
    _check(h, load().db_add_tether_bond_type(h, k_b, l_min, l_c1, l_c0, l_max, ctypes.byref(i)))
    return i.value


def db_set_reaction_melting(h, reaction, lam, T_melt, k_on_melt, k_off_melt):
    _check(h, load().db_set_reaction_melting(h, reaction, lam, T_melt, k_on_melt, k_off_melt))


def db_set_reaction_slip(h, reaction, a):
    _check(h, load().db_set_reaction_slip(h, reaction, a))


def db_set_temperature(h, kT):
    _check(h, load().db_set_temperature(h, kT))


def db_add_static_bonds(h, pairs, bond_types):
    p, pp = _buf(np.asarray(pairs).reshape(-1, 2), np.uint32)
    b, bp = _buf(np.asarray(bond_types).reshape(-1), np.uint32)
    _check(h, load().db_add_static_bonds(h, pp, bp, len(b)))


def make_reaction(type_a, type_b, bond_type, r_min, r_max, k_on=math.nan, k_off=math.nan,
                  epsilon=math.nan, p_on0=math.nan, self_avoid=-1):
    sa = -1 if self_avoid is None else int(self_avoid)
    return ReactionDesc(type_a, type_b, bond_type, r_min, r_max, k_on, k_off, epsilon, p_on0, sa)


def db_add_reaction(h, desc):
    i = _U32()
    _check(h, load().db_add_reaction(h, ctypes.byref(desc), ctypes.byref(i)))
    return i.value


def db_set_integrator(h, dt, kT, gamma, sweep_period, kt_source=DB_KT_SETPOINT):
    _check(h, load().db_set_integrator(h, dt, kT, gamma, sweep_period, kt_source))


def db_set_cell_capacity(h, slots):
    _check(h, load().db_set_cell_capacity(h, slots))


def db_set_step_shape(h, threads_per_particle, list_batch=0):
    _check(h, load().db_set_step_shape(h, threads_per_particle, list_batch))


def db_get_step_shape(h):
    """(threads per particle, list batch) of the step kernel."""
    t, q = _U32(), _U32()
    _check(h, load().db_get_step_shape(h, ctypes.byref(t), ctypes.byref(q)))
    return int(t.value), int(q.value)


def db_set_neighbor_list(h, skin=-1.0, max_neighbors=0):
    _check(h, load().db_set_neighbor_list(h, skin, max_neighbors))


def db_set_matching(h, grid_rounds=1, lds_limit=256):
    _check(h, load().db_set_matching(h, grid_rounds, lds_limit))


def db_validate(h):
    _check(h, load().db_validate(h))


def db_get_reaction(h, rid):
    d = ReactionDesc()
    pon, poff = _D(), _D()
    _check(h, load().db_get_reaction(h, rid, ctypes.byref(d), ctypes.byref(pon), ctypes.byref(poff)))
    return d, pon.value, poff.value


def db_commit(h):
    _check(h, load().db_commit(h))


def db_step(h, n_steps):
    _check(h, load().db_step(h, n_steps))


def _batch_raise(st, hs):
    # the failing system's message is in its own handle; report the first one
    for h in hs:
        msg = load().db_last_error(h)
        if msg:
            raise DybondError(st, msg.decode())
    raise DybondError(st, "")


def _plan_struct(plan):
    """A plan given as a list of (n_max, threads) classes, ascending n_max."""
    p = BatchPlan()
    p.n_classes = len(plan)                 # more than BATCH_MAX_CLASSES: the library rejects it
    for k, (n_max, threads) in enumerate(plan[:BATCH_MAX_CLASSES]):
        p.n_max[k] = min(int(n_max), 0xFFFFFFFF)
        p.threads[k] = int(threads)
    return p


def _plan_list(p):
    return [(int(p.n_max[k]), int(p.threads[k])) for k in range(p.n_classes)]


def db_step_batch(handles, n_steps):
    """Advance several committed systems (handles) by n_steps each in one
    chain of batched launches per size class, under the stored plan; bitwise equal
    to db_step on each."""
    hs = list(handles)
    arr = (ctypes.c_void_p * len(hs))(*hs)
    st = load().db_step_batch(arr, len(hs), n_steps)
    if st != 0:
        _batch_raise(st, hs)


def db_step_batch_plan(handles, n_steps, plan):
    """db_step_batch under an explicit plan [(n_max, threads), ...]."""
    hs = list(handles)
    arr = (ctypes.c_void_p * len(hs))(*hs)
    p = _plan_struct(plan)
    st = load().db_step_batch_plan(arr, len(hs), n_steps, ctypes.byref(p))
    if st != 0:
        _batch_raise(st, hs)


def db_set_batch_plan(device, plan):
    """Store the device's batch plan (None restores the default)."""
    p = None if plan is None else ctypes.byref(_plan_struct(plan))
    st = load().db_set_batch_plan(device, p)
    if st != 0:
        raise DybondError(st, "db_set_batch_plan")


def db_get_batch_plan(device):
    p = BatchPlan()
    st = load().db_get_batch_plan(device, ctypes.byref(p))
    if st != 0:
        raise DybondError(st, "db_get_batch_plan")
    return _plan_list(p)


def db_batch_autotune(handles, trial_steps):
    """Tune the device's batch plan on these systems; returns (plan,
    steps_done, trial times in ms).  The systems advance by steps_done."""
    hs = list(handles)
    arr = (ctypes.c_void_p * len(hs))(*hs)
    p = BatchPlan()
    done = _U64(0)
    ms = np.zeros(32, dtype=np.float64)                  # at most 1 + 4 x 5 timed trials
    st = load().db_batch_autotune(arr, len(hs), trial_steps, ctypes.byref(p), ctypes.byref(done), ms.ctypes.data,
                                  len(ms))
    if st != 0:
        _batch_raise(st, hs)
    n_timed = int(done.value) // trial_steps - 1          # every trial but the first is timed
    return _plan_list(p), int(done.value), ms[:max(0, n_timed)].tolist()


def db_sweep_frozen(h, step_key):
    _check(h, load().db_sweep_frozen(h, step_key))


def db_set_state(h, step, pos, vel, dyn_pairs=None, dyn_bond_types=None):
    p, pp = _buf(pos, np.float32)
    v, vp = _buf(vel, np.float32)
    pairs = np.zeros((0, 2), np.uint32) if dyn_pairs is None else np.asarray(dyn_pairs).reshape(-1, 2)
    bts = np.zeros(0, np.uint32) if dyn_bond_types is None else np.asarray(dyn_bond_types).reshape(-1)
    a, ap = _buf(pairs, np.uint32)
    b, bp = _buf(bts, np.uint32)
    _check(h, load().db_set_state(h, step, pp, vp, ap, bp, len(b)))


def db_save_checkpoint(h):
    """The system's checkpoint as bytes (size query, then the copy)."""
    size = _U64()
    st = load().db_save_checkpoint(h, None, 0, ctypes.byref(size))
    if st not in (DB_OK, DB_ETRUNC):
        _check(h, st)
    buf = ctypes.create_string_buffer(size.value)
    _check(h, load().db_save_checkpoint(h, ctypes.cast(buf, _P), size.value, ctypes.byref(size)))
    return buf.raw[:size.value]


def db_load_checkpoint(h, data):
    buf = ctypes.create_string_buffer(bytes(data), len(data))
    _check(h, load().db_load_checkpoint(h, ctypes.cast(buf, _P), len(data)))


def db_read_positions(h, n, with_images=False):
    pos = np.empty((n, 3), np.float32)
    img = np.empty((n, 3), np.int32) if with_images else None
    _check(h, load().db_read_positions(h, pos.ctypes.data_as(_P),
                                       img.ctypes.data_as(_P) if with_images else None))
    return (pos, img) if with_images else pos


def db_read_velocities(h, n):
    v = np.empty((n, 3), np.float32)
    _check(h, load().db_read_velocities(h, v.ctypes.data_as(_P)))
    return v


def db_read_forces(h, n):
    f = np.empty((n, 3), np.float32)
    _check(h, load().db_read_forces(h, f.ctypes.data_as(_P)))
    return f


def _read_bond_table(h, fn):
    cnt = _U64()
    st = fn(h, None, None, 0, ctypes.byref(cnt))
    if st not in (DB_OK, DB_ETRUNC):
        _check(h, st)
    m = cnt.value
    pairs = np.empty((m, 2), np.uint32)
    bts = np.empty(m, np.uint32)
    if m:
        _check(h, fn(h, pairs.ctypes.data_as(_P), bts.ctypes.data_as(_P), m, ctypes.byref(cnt)))
    return np.concatenate([pairs, bts[:, None]], axis=1).reshape(-1, 3)


def db_read_bonds(h):
    """Dynamic bonds as an (m, 3) uint32 array (tag_lo, tag_hi, bond_type)."""
    return _read_bond_table(h, load().db_read_bonds)


def db_read_bonds_noalloc(h):
    """db_read_bonds through the library's fixed device staging array (no
    device allocation inside the call)."""
    return _read_bond_table(h, load().db_read_bonds_noalloc)


def db_read_sweep_events(h, which):
    """Bonds formed (which = DB_EVENT_FORMED) or broken (DB_EVENT_BROKEN) by
    the last sweep: ((m, 3) uint32 array (tag_lo, tag_hi, bond_type) sorted,
    step key of that sweep, NO_SWEEP if none has run)."""
    cnt, step = _U64(), _U64()
    st = load().db_read_sweep_events(h, which, None, None, 0, ctypes.byref(cnt), ctypes.byref(step))
    if st not in (DB_OK, DB_ETRUNC):
        _check(h, st)
    m = cnt.value
    pairs = np.empty((m, 2), np.uint32)
    bts = np.empty(m, np.uint32)
    if m:
        _check(h, load().db_read_sweep_events(h, which, pairs.ctypes.data_as(_P), bts.ctypes.data_as(_P), m,
                                              ctypes.byref(cnt), ctypes.byref(step)))
    return np.concatenate([pairs, bts[:, None]], axis=1).reshape(-1, 3), step.value


def db_read_observables(h):
    o = Observables()
    _check(h, load().db_read_observables(h, ctypes.byref(o)))
    R = o.n_reactions
    return {"step": o.step, "n_bonds": np.array(o.n_bonds[:R]), "attempts": np.array(o.attempts[:R]),
            "forms": np.array(o.forms[:R]), "breaks": np.array(o.breaks[:R]),
            "bonded_fraction": np.array(o.bonded_fraction[:R]),
            "largest_cluster_fraction": o.largest_cluster_fraction,
            "PE": o.pe, "KE": o.ke, "T_kin": o.t_kin}


def db_bond_reference(h):
    _check(h, load().db_bond_reference(h))


def db_bond_correlation(h):
    """(reference bonds, reference bonds present now)."""
    a, b = _U64(), _U64()
    _check(h, load().db_bond_correlation(h, ctypes.byref(a), ctypes.byref(b)))
    return int(a.value), int(b.value)


def db_bond_multiplicity(h, length=8):
    """(hist of molecule pairs by number of joining bonds, bonded pairs,
    bonds inside one molecule)."""
    hist = np.zeros(length, dtype=np.uint64)
    pairs, intra = _U64(), _U64()
    _check(h, load().db_bond_multiplicity(h, hist.ctypes.data, length, ctypes.byref(pairs), ctypes.byref(intra)))
    return hist.astype(np.int64), int(pairs.value), int(intra.value)


def db_cluster_sizes(h, length=64):
    """(hist of clusters by size, number of clusters)."""
    hist = np.zeros(length, dtype=np.uint64)
    n = _U64()
    _check(h, load().db_cluster_sizes(h, hist.ctypes.data, length, ctypes.byref(n)))
    return hist.astype(np.int64), int(n.value)


def db_read_positions_device(h, dev_ptr, stream=None):
    """Positions (3 n floats, tag order) into device memory at dev_ptr (an
    integer address, e.g. tensor.data_ptr()), enqueued on `stream` (an
    integer hipStream_t, e.g. torch.cuda.current_stream().cuda_stream)."""
    _check(h, load().db_read_positions_device(h, dev_ptr, stream))


def db_read_velocities_device(h, dev_ptr, stream=None):
    _check(h, load().db_read_velocities_device(h, dev_ptr, stream))


def db_read_forces_device(h, dev_ptr, stream=None):
    _check(h, load().db_read_forces_device(h, dev_ptr, stream))


def db_read_list_builds(h):
    c = _U64()
    _check(h, load().db_read_list_builds(h, ctypes.byref(c)))
    return c.value


def db_get_step(h):
    return int(load().db_get_step(h))


def db_last_error(h):
    m = load().db_last_error(h)
    return m.decode() if m else ""


def db_set_stream(h, stream_ptr):
    _check(h, load().db_set_stream(h, stream_ptr))


def db_kernel_timing(h, enable):
    _check(h, load().db_kernel_timing(h, 1 if enable else 0))


def db_read_kernel_time(h, kernel):
    n, ms = _U64(), _D()
    _check(h, load().db_read_kernel_time(h, kernel.encode(), ctypes.byref(n), ctypes.byref(ms)))
    return n.value, ms.value


# ---------------------------------------------------------------- surrogate network
def _mcheck(net, status):
    if status != DB_OK:
        msg = load().db_mlp_last_error(net)
        raise DybondError(status, msg.decode() if msg else "")


def _f32(a, cols):
    return np.ascontiguousarray(np.asarray(a, dtype=np.float32).reshape(-1, cols))


def db_mlp_create(batch_max, device=0):
    h = _P()
    st = load().db_mlp_create(batch_max, device, ctypes.byref(h))
    if st != DB_OK:
        raise DybondError(st, "db_mlp_create")
    return h.value


def db_mlp_destroy(net):
    load().db_mlp_destroy(net)


def db_mlp_set_params(net, params):
    p = np.ascontiguousarray(np.asarray(params, dtype=np.float32).reshape(-1))
    _mcheck(net, load().db_mlp_set_params(net, p.ctypes.data, p.size))


def db_mlp_get_params(net):
    p = np.zeros(MLP_PARAMS, dtype=np.float32)
    _mcheck(net, load().db_mlp_get_params(net, p.ctypes.data, p.size))
    return p


def db_mlp_predict(net, x):
    x = _f32(x, 4)
    y = np.zeros((len(x), 2), dtype=np.float32)
    _mcheck(net, load().db_mlp_predict(net, x.ctypes.data, len(x), y.ctypes.data))
    return y


def db_mlp_loss_grad(net, x, t):
    x, t = _f32(x, 4), _f32(t, 2)
    loss = ctypes.c_float()
    g = np.zeros(MLP_PARAMS, dtype=np.float32)
    _mcheck(net, load().db_mlp_loss_grad(net, x.ctypes.data, t.ctypes.data, len(x), ctypes.byref(loss), g.ctypes.data))
    return float(loss.value), g


def db_mlp_train(net, x, t, batch, epochs, lr, seed=1):
    x, t = _f32(x, 4), _f32(t, 2)
    loss = ctypes.c_float()
    _mcheck(net, load().db_mlp_train(net, x.ctypes.data, t.ctypes.data, len(x), batch, epochs, lr, seed,
                                     ctypes.byref(loss)))
    return float(loss.value)


def db_mlp_last_error(net):
    msg = load().db_mlp_last_error(net)
    return msg.decode() if msg else ""


# ---------------------------------------------------------------- convenience
class System:
    """Owns one handle; ``from_workload`` replays the set-up calls for a
    workload built by :mod:`paper_2609_21204_amd.inputs`."""

    def __init__(self, n, n_types, box_L, seed, device=0):
        self.n = int(n)
        self.h = db_create(n, n_types, box_L, seed, device)

    @classmethod
    def from_workload(cls, w, device=0, commit=True, kt_source=DB_KT_SETPOINT, skin=None, max_neighbors=0,
                      matching=None):
        s = cls(w.n, len(w.types), w.L, w.seed, device)
        if skin is not None or max_neighbors:
            db_set_neighbor_list(s.h, -1.0 if skin is None else skin, max_neighbors)
        if matching is not None:
            db_set_matching(s.h, *matching)
        for t, (val, sig, eps, m) in enumerate(w.types):
            db_set_type(s.h, t, val, sig, eps, m)
        db_set_particles(s.h, w.pos, w.vel, w.type_id)
        for bt in w.bond_types:
            if bt[0] == DB_BOND_TETHER:                # (kind, k_b, l_min, l_c1, l_c0, l_max)
                db_add_tether_bond_type(s.h, *bt[1:])
            else:
                db_add_bond_type(s.h, *bt)
        if len(w.static_pairs):
            db_add_static_bonds(s.h, w.static_pairs, w.static_types)
        for a, r in enumerate(w.reactions):
            r = dict(r)
            melt, slip = r.pop("melt", None), r.pop("slip", None)
            db_add_reaction(s.h, make_reaction(**r))
            if melt is not None:
                db_set_reaction_melting(s.h, a, *melt)
            if slip is not None:
                db_set_reaction_slip(s.h, a, slip)
        db_set_integrator(s.h, w.dt, w.kT, w.gamma, w.period, kt_source)
        if commit:
            db_commit(s.h)
        return s

    def close(self):
        if self.h:
            db_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def __enter__(self):
        return self

    def __exit__(self, *a):
        self.close()

    # marshalling shortcuts
    def step(self, n):
        db_step(self.h, n)

    def sweep_frozen(self, key):
        db_sweep_frozen(self.h, key)

    def positions(self, with_images=False):
        return db_read_positions(self.h, self.n, with_images)

    def velocities(self):
        return db_read_velocities(self.h, self.n)

    def forces(self):
        return db_read_forces(self.h, self.n)

    def bonds(self):
        return db_read_bonds(self.h)

    def sweep_events(self, which):
        return db_read_sweep_events(self.h, which)

    def observables(self):
        return db_read_observables(self.h)

    def set_state(self, step, pos, vel, pairs=None, bts=None):
        db_set_state(self.h, step, pos, vel, pairs, bts)

    def save_checkpoint(self):
        return db_save_checkpoint(self.h)

    def load_checkpoint(self, data):
        db_load_checkpoint(self.h, data)

    @property
    def step_count(self):
        return db_get_step(self.h)
