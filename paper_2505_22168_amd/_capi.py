"""ctypes view of the C ABI in include/gmnn.h (argument marshalling only)."""
from __future__ import annotations

import ctypes as C
import os

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libgmnn.so")

GMNN_OK = 0
GMNN_ERR_INVALID_ARG = -1
GMNN_ERR_CAPACITY = -2
GMNN_ERR_UNSUPPORTED = -3
GMNN_ERR_HIP = -4
GMNN_ERR_DEVICE_FLAG = -5
GMNN_ERR_WORKSPACE = -6
GMNN_ERR_SCRATCH_LIMIT = -7
GMNN_OP_FEATURES = 3
GMNN_NOALLOC_SCRATCH_BYTES = 64 << 20

GMNN_FLAG_CAPACITY = 1
GMNN_FLAG_NONFINITE = 2
GMNN_FLAG_COINCIDENT = 4
GMNN_FLAG_ROW_TOO_LONG = 8
GMNN_FLAG_SHIFT_RANGE = 16
GMNN_MAX_ROW = 1024

GMNN_PREC_FP32 = 0
GMNN_PREC_BF16 = 1
GMNN_WANT_STRESS = 2
GMNN_WANT_FORCE_VAR = 4
GMNN_SYNC = 8
GMNN_BACKWARD_LANES16 = 16
GMNN_BACKWARD_PER_HEAD = 32
GMNN_HEADS_TILE = 64
GMNN_LOSS_MSE, GMNN_LOSS_NLL, GMNN_LOSS_CRPS = 0, 1, 2
GMNN_GROUP_EMBEDDING, GMNN_GROUP_NN, GMNN_GROUP_SCALE, GMNN_GROUP_SHIFT = 0, 1, 2, 3
GMNN_LR_CONSTANT, GMNN_LR_LINEAR, GMNN_LR_COSINE = 0, 1, 2

GMNN_SCHEDULE_AUTO = 0
GMNN_SCHEDULE_FUSED = 1
GMNN_SCHEDULE_SPLIT = 2
GMNN_READOUT_AUTO = 0
GMNN_READOUT_TILE = 1
GMNN_READOUT_STREAM = 2

GMNN_OP_NEIGHBORS = 0
GMNN_OP_ENERGY_FORCES = 1
GMNN_OP_BACKWARD = 2

vp = C.c_void_p


class gmnn_system(C.Structure):
    _fields_ = [("n_structs", C.c_int32), ("n_atoms", C.c_int32),
                ("atom_ptr", vp), ("atom_ptr_host", vp), ("pos", vp), ("species", vp),
                ("cell", vp), ("cell_host", vp), ("pbc", vp), ("pbc_host", vp)]


class gmnn_neighbors(C.Structure):
    _fields_ = [("capacity", C.c_int64), ("row_ptr", vp), ("j", vp), ("shift", vp), ("rev", vp),
                ("atom_struct", vp), ("n_pairs", vp), ("status", vp), ("cutoff", C.c_float)]


class gmnn_model(C.Structure):
    _fields_ = [("n_species", C.c_int32), ("n_radial", C.c_int32), ("n_basis", C.c_int32),
                ("hidden1", C.c_int32), ("hidden2", C.c_int32), ("n_heads", C.c_int32),
                ("r_min", C.c_float), ("r_cut", C.c_float), ("gamma", C.c_float), ("psi_scale", C.c_float),
                ("beta", vp), ("W1", vp), ("b1", vp), ("W2", vp), ("b2", vp), ("W3", vp), ("b3", vp),
                ("scale", vp), ("shift", vp), ("packed", vp), ("basis", C.c_int32)]


GMNN_BASIS_GAUSSIAN = 0
GMNN_BASIS_BESSEL = 1


class gmnn_udd(C.Structure):
    _fields_ = [("A", C.c_float), ("B", C.c_float), ("bias_energy", vp)]


class gmnn_param_grads(C.Structure):
    _fields_ = [(k, vp) for k in ("beta", "W1", "b1", "W2", "b2", "W3", "b3", "scale", "shift")]


class gmnn_md(C.Structure):
    _fields_ = [("dt", C.c_float), ("skin", C.c_float), ("inv_mass", vp), ("vel", vp), ("forces", vp),
                ("energy", vp), ("ref_pos", vp), ("disp", vp), ("udd", vp), ("var_every", C.c_int32),
                ("force_var", vp), ("energy_var", vp)]


class gmnn_plan(C.Structure):
    _fields_ = [("schedule", C.c_int32), ("lanes_per_atom", C.c_int32), ("readout", C.c_int32),
                ("tile_atoms", C.c_int32)]

    FIELDS = ("schedule", "lanes_per_atom", "readout", "tile_atoms")

    @classmethod
    def of(cls, plan) -> "gmnn_plan":
        """From a dict with these field names (missing: 0) or a tuple in field order."""
        if isinstance(plan, dict):
            plan = tuple(int(plan.get(k, 0)) for k in cls.FIELDS)
        plan = tuple(int(v) for v in plan) + (0,) * (len(cls.FIELDS) - len(plan))
        return cls(*plan)

    def as_dict(self) -> dict:
        return {k: int(getattr(self, k)) for k in self.FIELDS}


class gmnn_tune_entry(C.Structure):
    _fields_ = [("plan", gmnn_plan), ("median_us", C.c_float), ("min_us", C.c_float)]


class gmnn_outputs(C.Structure):
    _fields_ = [("energy", vp), ("forces", vp), ("stress", vp), ("energy_var", vp),
                ("force_var", vp), ("atomic_energy", vp), ("energy_mean", vp), ("status", vp),
                ("forces_heads", vp)]


class gmnn_loss(C.Structure):
    _fields_ = [("energy_kind", C.c_int32), ("force_kind", C.c_int32), ("energy_per_atom", C.c_int32),
                ("reserved", C.c_int32), ("w_energy", C.c_double), ("w_force", C.c_double),
                ("var_floor", C.c_double)]


class gmnn_adam(C.Structure):
    _fields_ = [("lr", C.c_double * 4), ("beta1", C.c_double), ("beta2", C.c_double), ("eps", C.c_double),
                ("step", C.c_int64)]


class gmnn_lr_schedule(C.Structure):
    _fields_ = [("kind", C.c_int32), ("reserved", C.c_int32), ("total_steps", C.c_int64),
                ("end_factor", C.c_double), ("period", C.c_int64), ("decay_factor", C.c_double)]


EXPORTS = {
    "gmnn_loss_workspace_bytes": (C.c_size_t, [C.POINTER(gmnn_system)]),
    "gmnn_ensemble_loss": (C.c_int32, [C.POINTER(gmnn_loss), C.POINTER(gmnn_system), C.c_int32, vp, vp, vp, vp,
                                       vp, vp, vp, vp, C.c_size_t, vp]),
    "gmnn_adam_step": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_param_grads), C.POINTER(gmnn_param_grads),
                                   C.POINTER(gmnn_param_grads), C.POINTER(gmnn_adam), vp]),
    "gmnn_lr_factor": (C.c_double, [C.POINTER(gmnn_lr_schedule), C.c_int64]),
    "gmnn_status_string": (C.c_char_p, [C.c_int32]),
    "gmnn_num_features": (C.c_int32, [C.c_int32]),
    "gmnn_model_packed_bytes": (C.c_size_t, [C.POINTER(gmnn_model)]),
    "gmnn_model_prepare": (C.c_int32, [C.POINTER(gmnn_model), vp]),
    "gmnn_workspace_bytes": (C.c_size_t, [C.c_int32, C.POINTER(gmnn_model), C.POINTER(gmnn_system),
                                          C.POINTER(gmnn_neighbors), C.c_uint32]),
    "gmnn_neighbors_workspace_bytes": (C.c_size_t, [C.POINTER(gmnn_system), C.c_float, C.c_float]),
    "gmnn_build_neighbors": (C.c_int32, [C.POINTER(gmnn_system), C.c_float, C.c_float,
                                         C.POINTER(gmnn_neighbors), C.c_uint32, vp, C.c_size_t, vp]),
    "gmnn_energy_forces_udd": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system), C.POINTER(gmnn_neighbors),
                                           C.c_uint32, C.POINTER(gmnn_plan), C.POINTER(gmnn_udd),
                                           C.POINTER(gmnn_outputs), vp, C.c_size_t, vp]),
    "gmnn_last_layer_features": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system),
                                             C.POINTER(gmnn_neighbors), C.c_uint32, vp, vp, C.c_size_t, vp]),
    "gmnn_select_workspace_bytes": (C.c_size_t, [C.c_int64]),
    "gmnn_select_max_distance": (C.c_int32, [vp, C.c_int64, C.c_int32, vp, C.c_int64, C.c_int32, vp, vp,
                                             C.c_size_t, vp]),
    "gmnn_energy_forces_noalloc": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system),
                                               C.POINTER(gmnn_neighbors), C.c_uint32, C.POINTER(gmnn_outputs), vp]),
    "gmnn_energy_forces": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system), C.POINTER(gmnn_neighbors),
                                       C.c_uint32, C.POINTER(gmnn_outputs), vp, C.c_size_t, vp]),
    "gmnn_resolve_plan": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system), C.c_uint32,
                                      C.POINTER(gmnn_plan), C.POINTER(gmnn_plan)]),
    "gmnn_uses_fused_path": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system), C.c_uint32]),
    "gmnn_energy_forces_plan": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system),
                                            C.POINTER(gmnn_neighbors), C.c_uint32, C.POINTER(gmnn_plan),
                                            C.POINTER(gmnn_outputs), vp, C.c_size_t, vp]),
    "gmnn_energy_forces_timed": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system),
                                             C.POINTER(gmnn_neighbors), C.c_uint32, C.POINTER(gmnn_plan),
                                             C.POINTER(gmnn_outputs), vp, C.c_size_t, vp, vp]),
    "gmnn_autotune": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system), C.POINTER(gmnn_neighbors),
                                  C.c_uint32, C.POINTER(gmnn_outputs), vp, C.c_size_t, vp, C.c_int32,
                                  C.POINTER(gmnn_plan), C.POINTER(gmnn_tune_entry), C.c_int32,
                                  C.POINTER(C.c_int32)]),
    "gmnn_backward": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system), C.POINTER(gmnn_neighbors),
                                  vp, vp, C.c_uint32, C.POINTER(gmnn_param_grads), vp, vp, C.c_size_t, vp]),
    "gmnn_md_workspace_bytes": (C.c_size_t, [C.POINTER(gmnn_model), C.POINTER(gmnn_system),
                                             C.POINTER(gmnn_neighbors), C.c_uint32]),
    "gmnn_md_init": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system), C.POINTER(gmnn_neighbors),
                                 C.POINTER(gmnn_md), C.c_uint32, vp, C.c_size_t, vp]),
    "gmnn_md_steps": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system), C.POINTER(gmnn_neighbors),
                                  C.POINTER(gmnn_md), C.c_uint32, C.c_int32, vp, C.c_size_t, vp]),
    "gmnn_md_graph_create": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system), C.POINTER(gmnn_neighbors),
                                         C.POINTER(gmnn_md), C.c_uint32, C.c_int32, vp, C.c_size_t,
                                         C.POINTER(C.c_void_p)]),
    "gmnn_md_graph_launch": (C.c_int32, [vp, vp]),
    "gmnn_md_graph_destroy": (None, [vp]),
    "gmnn_energy_forces_graph_create": (C.c_int32, [C.POINTER(gmnn_model), C.POINTER(gmnn_system),
                                                    C.POINTER(gmnn_neighbors), C.c_uint32, C.POINTER(gmnn_plan),
                                                    C.POINTER(gmnn_outputs), vp, C.c_size_t, C.c_int32,
                                                    C.POINTER(C.c_void_p)]),
    "gmnn_graph_launch": (C.c_int32, [vp, vp]),
    "gmnn_graph_destroy": (None, [vp]),
}

_lib = None


def load(path: str = LIB_PATH):
    """Load libgmnn.so (raises if it has not been built)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(path):
        raise ImportError(f"{path} is missing: build it with `python -m paper_2505_22168_amd.build`")
    lib = C.CDLL(path)
    for name, (res, args) in EXPORTS.items():
        fn = getattr(lib, name)
        fn.restype = res
        fn.argtypes = args
    _lib = lib
    return lib


class GMNNError(RuntimeError):
    def __init__(self, status: int, where: str):
        msg = load().gmnn_status_string(status).decode()
        super().__init__(f"{where}: status {status} ({msg})")
        self.status = status


def check(status: int, where: str):
    if status != GMNN_OK:
        raise GMNNError(status, where)
