"""ctypes loader for librtssa.so (argument marshalling only).

The library is built in-tree by ``paper_2103_00405_amd/build.py``.  There is
no fallback: if the shared object is missing or fails to load, every entry
point raises.
"""
import ctypes as C
import os

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.environ.get("RTSSA_LIB") or os.path.join(HERE, "librtssa.so")

_lib = None

vp = C.c_void_p
i32, i64, u32, u64, f64 = C.c_int32, C.c_int64, C.c_uint32, C.c_uint64, C.c_double


class Stats(C.Structure):
    _fields_ = [("firings", u64), ("near_ties", u64), ("clamps", u64), ("slow_logs", u64),
                ("status_count", u64 * 4), ("kernel_ms", f64), ("mapping", i32),
                ("block", i32), ("grid", i32), ("bad_input", i32)]

    def as_dict(self):
        return dict(firings=int(self.firings), near_ties=int(self.near_ties),
                    clamps=int(self.clamps), slow_logs=int(self.slow_logs),
                    status_count=[int(x) for x in self.status_count],
                    kernel_ms=float(self.kernel_ms), mapping=int(self.mapping),
                    block=int(self.block), grid=int(self.grid), bad_input=int(self.bad_input))


class Options(C.Structure):
    _fields_ = [("max_firings", u64), ("mapping", i32), ("block", i32), ("grid", i32),
                ("method", i32), ("workspace", vp), ("workspace_bytes", u64)]


class BatchItem(C.Structure):
    _fields_ = [("net", vp), ("x0", vp), ("x0_per_traj", i32), ("G", i32), ("t_end", f64),
                ("sample_t", vp), ("net_id", u32), ("method", i32), ("traj_offset", u64),
                ("R", i64), ("samples", vp), ("s_stride_r", i64), ("s_stride_g", i64),
                ("s_stride_n", i64), ("n_out", vp), ("T_out", vp), ("x_final", vp),
                ("t_last", vp), ("status", vp), ("seq_hash", vp), ("tie_step", vp),
                ("weight", f64)]


SIGNATURES = {
    "rtssa_last_error": (C.c_char_p, []),
    "rtssa_version": (C.c_char_p, []),
    "rtssa_network_create": (C.c_int, [i32, i32, vp, vp, vp, vp, vp, vp, vp, C.POINTER(vp)]),
    "rtssa_network_destroy": (C.c_int, [vp]),
    "rtssa_network_set_rates": (C.c_int, [vp, vp]),
    "rtssa_network_set_schedule": (C.c_int, [vp, i32, vp, vp]),
    "rtssa_network_info": (C.c_int, [vp, vp, vp, vp, vp]),
    "rtssa_simulate": (C.c_int, [vp, vp, i32, f64, vp, i32, u64, u32, u64, i64, vp, i64, i64,
                                 i64, vp, vp, vp, vp, vp, vp, vp, C.POINTER(Options), vp,
                                 C.POINTER(Stats)]),
    "rtssa_simulate_noalloc": (C.c_int, [vp, vp, i32, f64, vp, i32, u64, u32, u64, i64, vp, i64,
                                         i64, i64, vp, vp, vp, vp, vp, vp, vp,
                                         C.POINTER(Options), vp, C.POINTER(Stats)]),
    "rtssa_workspace_size": (C.c_int, [vp, i64, C.POINTER(Options), C.POINTER(C.c_size_t)]),
    "rtssa_score_grad_workspace_size": (C.c_int, [i64, i32, C.POINTER(C.c_size_t)]),
    "rtssa_score_grad": (C.c_int, [vp, vp, vp, i64, i32, i32, vp, vp, vp, u64, vp]),
    "rtssa_batch_create": (C.c_int, [C.POINTER(BatchItem), i32, C.POINTER(Options), C.c_char_p,
                                     C.POINTER(vp)]),
    "rtssa_batch_run": (C.c_int, [vp, u64, i32, vp, C.POINTER(Stats)]),
    "rtssa_batch_info": (C.c_int, [vp, i32, vp, vp, vp, vp, vp]),
    "rtssa_batch_class_items": (C.c_int, [vp, i32, vp, i32, C.POINTER(i32)]),
    "rtssa_batch_destroy": (C.c_int, [vp]),
    "rtssa_autotune": (C.c_int, [C.POINTER(BatchItem), i32, i32, C.c_char_p, vp]),
    "rtssa_debug_neglog": (C.c_int, [vp, vp, vp, i64, i32, vp]),
    "rtssa_debug_neglog_host": (f64, [u64, i32, C.POINTER(i32)]),
    "rtssa_debug_recip": (i32, [vp, vp, i64, vp]),
    "rtssa_debug_neglog_quick_host": (i32, [u64, C.POINTER(f64)]),
    "rtssa_debug_neglog_fast_host": (None, [u64, C.POINTER(f64), C.POINTER(f64)]),
    "rtssa_debug_philox": (C.c_int, [vp, u32, u32, vp, i64, vp]),
    "rtssa_debug_select": (C.c_int, [vp, i32, i64, i32, i32, vp, vp, vp, vp, vp]),
    "rtssa_debug_philox_host": (None, [vp, u32, u32, vp]),
}


class RtssaError(RuntimeError):
    def __init__(self, code, msg):
        super().__init__("rtssa error %d: %s" % (code, msg))
        self.code = code


def lib():
    """Load librtssa.so; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError("librtssa.so is not built; run paper_2103_00405_amd/build.py "
                               "(or __graft_entry__.build()) first")
        L = C.CDLL(LIB_PATH)
        for name, (res, args) in SIGNATURES.items():
            fn = getattr(L, name)
            fn.restype = res
            fn.argtypes = args
        _lib = L
    return _lib


def check(rc):
    if rc != 0:
        raise RtssaError(rc, lib().rtssa_last_error().decode())
    return rc
