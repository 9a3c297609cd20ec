"""What the library's own rules say about a call, for tests that have to reach one kernel or one kind of plan: host code of the built
library, which needs no GPU."""
import ctypes as C

from paper_2502_02406_amd import binding as B

N_CU = 256                                           # compute units of the device that the tests run on


class _Dims(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("B", "Hq", "Hkv", "Sq", "Skv", "D", "G")] + \
               [(n, C.c_long) for n in ("q_sb", "q_sh", "q_ss", "kv_sb", "kv_sh", "kv_ss")] + [("scale", C.c_float)]


class _Mask(C.Structure):
    _fields_ = [("allow", C.c_void_p)] + [(n, C.c_int) for n in ("q_chunk", "kv_block", "n_q_chunks", "n_kv_blocks")] + \
               [("stride_b", C.c_long), ("stride_q", C.c_long)]


class _KvPlan(C.Structure):
    _fields_ = [("whole", C.c_int), ("parts", C.c_int), ("len", C.c_int)]


class _TailPlan(C.Structure):
    _fields_ = [("whole", C.c_int), ("parts", C.c_int)]


def _dims(B_, Hq, Hkv, Sq, Skv, D):
    return _Dims(B_, Hq, Hkv, Sq, Skv, D, Hq // Hkv, Hq * Sq * D, Sq * D, D, Hkv * Skv * D, Skv * D, D, D ** -0.5)


def dkdv_parts(*shape, masked=False):
    """(tiles of 256 keys of a head that have a workgroup to themselves, the most workgroups that share another) where there is room
    for as many as the plan wants."""
    f = B.load()._ZN3lvx14dkdv_bf16_planERKNS_4DimsEibl
    f.restype, f.argtypes = _KvPlan, [C.POINTER(_Dims), C.c_int, C.c_bool, C.c_long]
    p = f(C.byref(_dims(*shape)), N_CU, masked, 1 << 20)
    return p.whole, p.parts


def dkdv_is_short(*shape, q_chunk=0, kv_block=0):
    """Whether the kernel for key tiles of few steps takes the call, given that no tile is shared."""
    f = B.load()._ZN3lvx20bwd_dkdv_short_takesERKNS_4DimsERKNS_7MaskDevEi
    f.restype, f.argtypes = C.c_bool, [C.POINTER(_Dims), C.POINTER(_Mask), C.c_int]
    mode = 0 if q_chunk == 0 else 1 if q_chunk % 32 == 0 and kv_block % 256 == 0 else 2
    return f(C.byref(_dims(*shape)), C.byref(_Mask(None, max(q_chunk, 1), max(kv_block, 1), 1, 1, 0, 1)), mode)


def fwd_plan(*shape, running=False):
    """(row tiles of a K/V head that one workgroup takes, parts of the others) of the dense forward."""
    f = B.load()._ZN3lvx19fwd_bf16_dense_planERKNS_4DimsEiii
    f.restype, f.argtypes = _TailPlan, [C.POINTER(_Dims), C.c_int, C.c_int, C.c_int]
    p = f(C.byref(_dims(*shape)), N_CU, B.LVX_MAX_PARTS - running, 2 if shape[5] == 64 else 1)
    return p.whole, p.parts
