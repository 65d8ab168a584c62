"""The library's calls for torch tensors.  Function names and argument order follow
include/signsgd.h (ss_ prefix dropped).  Tensors are checked and unpacked by the native
module _marshal (csrc/marshal.cpp); load_library() is the plain ctypes handle of
libsignsgd.so for callers with raw pointers."""
import ctypes
import os

import torch

F32 = 0
BF16 = 1
MAX_WORKERS = 64

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libsignsgd.so")
_lib = None

_STATUS = {0: "SS_OK", -1: "SS_ERR_NULL", -2: "SS_ERR_BAD_M", -3: "SS_ERR_ALIGN",
           -4: "SS_ERR_DTYPE", -5: "SS_ERR_ARG", -6: "SS_ERR_HIP", -7: "SS_ERR_RANGE"}


class SignSGDError(RuntimeError):
    def __init__(self, call, status):
        self.status = status
        detail = ""
        if status == -6 and _lib is not None:
            detail = " (hipError_t %d)" % _lib.ss_last_hip_error()
        super().__init__("%s returned %s%s" % (call, _STATUS.get(status, status), detail))


def library_path():
    return _LIB_PATH


def load_library():
    """Load the built HIP library; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise ImportError(
                "%s is missing: build it with `python -m paper_1802_04434_amd.build` "
                "(there is no fallback path)" % _LIB_PATH)
        L = ctypes.CDLL(_LIB_PATH)
        vp, sz, i32, f32 = ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int, ctypes.c_float
        L.ss_packed_words.restype = sz
        L.ss_packed_words.argtypes = [sz]
        L.ss_packed_bytes.restype = sz
        L.ss_packed_bytes.argtypes = [sz]
        L.ss_last_hip_error.restype = i32
        L.ss_last_hip_error.argtypes = []
        L.ss_signum_pack.argtypes = [vp, i32, vp, f32, vp, sz, vp]
        L.ss_majority_vote.argtypes = [vp, i32, vp, sz, vp]
        L.ss_sign_apply.argtypes = [vp, vp, f32, sz, vp]
        L.ss_signum_vote_step.argtypes = [vp, i32, vp, i32, f32, f32, vp, vp, vp, sz, vp]
        L.ss_stream_copy.argtypes = [vp, vp, sz, vp]
        L.ss_warmup_length.restype = ctypes.c_long
        L.ss_warmup_length.argtypes = [f32]
        L.ss_signum_pack_warmup.argtypes = [vp, i32, vp, f32, vp, sz, vp]
        L.ss_vote_sum.argtypes = [vp, i32, vp, sz, vp]
        L.ss_sum_apply.argtypes = [vp, vp, f32, sz, vp]
        L.ss_signum_vote_step_ex.argtypes = [vp, i32, vp, i32, f32, f32, vp, vp, vp, vp, sz, ctypes.c_uint, vp]
        L.ss_step_scratch_bytes.restype = sz
        L.ss_step_scratch_bytes.argtypes = [i32, i32, i32, sz]
        L.ss_signum_vote_step_scratch.argtypes = [vp, i32, vp, i32, f32, f32, vp, vp, vp, vp, sz, sz, ctypes.c_uint, vp]
        L.ss_signum_vote_step_scratch.restype = i32
        L.ss_ternary_scratch_bytes.restype = sz
        L.ss_ternary_scratch_bytes.argtypes = [i32, i32, i32, sz]
        L.ss_signum_vote_step_ternary_scratch.argtypes = [vp, i32, vp, i32, f32, f32, i32, f32, vp, vp, vp, vp, sz, sz, vp]
        L.ss_signum_vote_step_ternary_scratch.restype = i32
        L.ss_welford_update.argtypes = [vp, i32, vp, vp, ctypes.c_uint64, sz, vp]
        L.ss_welford_sigma.argtypes = [vp, ctypes.c_uint64, vp, sz, vp]
        L.ss_density.argtypes = [vp, sz, vp, vp, vp]
        L.ss_density_workspace_bytes.restype = sz
        L.ss_density_workspace_bytes.argtypes = []
        L.ss_density_static.argtypes = [vp, sz, vp, vp]
        L.ss_density_static.restype = i32
        L.ss_signum_pack_ternary.argtypes = [vp, i32, vp, f32, f32, vp, vp, sz, vp]
        L.ss_quorum_vote.argtypes = [vp, vp, i32, i32, vp, vp, sz, vp]
        L.ss_ternary_apply.argtypes = [vp, vp, vp, f32, sz, vp]
        L.ss_signum_vote_step_ternary.argtypes = [vp, i32, vp, i32, f32, f32, i32, f32, vp, vp, vp, sz, vp]
        for name in ("ss_signum_pack_ternary", "ss_quorum_vote", "ss_ternary_apply",
                     "ss_signum_vote_step_ternary"):
            getattr(L, name).restype = i32
        for name in ("ss_welford_update", "ss_welford_sigma", "ss_density"):
            getattr(L, name).restype = i32
        for name in ("ss_signum_pack", "ss_majority_vote", "ss_sign_apply", "ss_signum_vote_step",
                     "ss_stream_copy", "ss_signum_pack_warmup", "ss_vote_sum", "ss_sum_apply",
                     "ss_signum_vote_step_ex"):
            getattr(L, name).restype = i32
        _lib = L
    return _lib


def packed_words(d):
    return load_library().ss_packed_words(d)


def packed_bytes(d):
    return load_library().ss_packed_bytes(d)


def last_hip_error():
    return load_library().ss_last_hip_error()


def new_bits(d, device="cuda"):
    """uninitialised packed / voted buffer for d coordinates (int32 storage)"""
    return torch.empty(packed_bytes(d) // 4, dtype=torch.int32, device=device)


_marshal = None


def _native():
    """the module that marshals torch tensors into the library; raises if it has not been built"""
    global _marshal
    if _marshal is None:
        load_library()
        from . import _marshal as module
        _marshal = module
    return _marshal


def _check(call, status):
    if status != 0:
        raise SignSGDError(call, status)


def signum_pack(g, m, beta, packed, d=None, stream=None):
    """ss_signum_pack: m <- beta m + (1-beta) g; packed <- bits of sign(m)
    (m None: bits of sign(g))."""
    _check("ss_signum_pack", (_marshal or _native()).signum_pack(g, m, beta, packed, d, stream, False))
    return packed


def signum_pack_warmup(g, m, beta, packed, d=None, stream=None):
    """ss_signum_pack_warmup: m updated as above, packed <- bits of sign(g)"""
    _check("ss_signum_pack_warmup", (_marshal or _native()).signum_pack(g, m, beta, packed, d, stream, True))
    return packed


def warmup_length(beta):
    """ss_warmup_length: Theorem 3's C(beta)"""
    c = load_library().ss_warmup_length(beta)
    if c < 0:
        raise SignSGDError("ss_warmup_length", c)
    return c


def vote_sum(packed, sums, d, stream=None):
    """ss_vote_sum: sums <- per-coordinate sum of the workers' signs (int8)"""
    _check("ss_vote_sum", (_marshal or _native()).vote_sum(packed, sums, d, stream))
    return sums


def sum_apply(x, sums, delta, d=None, stream=None):
    """ss_sum_apply: x <- x - delta * sums"""
    _check("ss_sum_apply", (_marshal or _native()).sum_apply(x, sums, delta, d, stream))
    return x


def majority_vote(packed, voted, d, stream=None):
    """ss_majority_vote: voted <- bits of sign(sum_w sign_w)"""
    _check("ss_majority_vote", (_marshal or _native()).majority_vote(packed, voted, d, stream))
    return voted


def sign_apply(x, bits, delta, d=None, stream=None):
    """ss_sign_apply: x <- x - delta * (+-1 from bits)"""
    _check("ss_sign_apply", (_marshal or _native()).sign_apply(x, bits, delta, d, stream))
    return x


STEP_DEFAULT = 0
STEP_WARMUP = 1
STEP_SUM_UPDATE = 2


def signum_vote_step(g, m, beta, delta, x, voted, packed_out=None, d=None, stream=None):
    """ss_signum_vote_step: the whole step for M = len(g) workers in one call.
    g: list of gradients; m: list of momentum buffers or None.
    A large step with momentum and without packed_out borrows up to 128 MiB from
    torch's caching allocator for the length of the call
    (ss_signum_vote_step_scratch).  It does so on torch's own streams, outside of
    capture, and while a gigabyte of device memory stays free beside it; otherwise
    it runs in one pass, with the same results.  The allocator keeps such a block
    for each stream until it needs the memory (torch.cuda.empty_cache)."""
    _check("ss_signum_vote_step", (_marshal or _native()).signum_vote_step(
        g, m, beta, delta, x, voted, packed_out, None, 0, d, stream))
    return voted


def signum_vote_step_ex(g, m, beta, delta, x, voted, packed_out=None, sums_out=None, flags=None, d=None,
                        stream=None):
    """ss_signum_vote_step_ex (flags None: the plain step); borrows memory as signum_vote_step does"""
    _check("ss_signum_vote_step_ex", (_marshal or _native()).signum_vote_step(
        g, m, beta, delta, x, voted, packed_out, sums_out, int(flags or 0), d, stream))
    return voted


def stream_copy(dst, src, nbytes, stream=None):
    """ss_stream_copy: measurement aid, dst <- src"""
    _check("ss_stream_copy", (_marshal or _native()).stream_copy(dst, src, nbytes, stream))


def welford_update(g, mean, m2, n, d=None, stream=None):
    """ss_welford_update: fold the n-th gradient (n counts from 1) into mean / m2"""
    _check("ss_welford_update", (_marshal or _native()).welford_update(g, mean, m2, n, d, stream))


def welford_sigma(m2, n, sigma, d=None, stream=None):
    """ss_welford_sigma: sigma <- sqrt(m2 / n)"""
    _check("ss_welford_sigma", (_marshal or _native()).welford_sigma(m2, n, sigma, d, stream))
    return sigma


def new_density_workspace(device="cuda"):
    """zero-filled workspace for ss_density (ss_density_workspace_bytes() bytes)"""
    return torch.zeros(load_library().ss_density_workspace_bytes() // 8, dtype=torch.int64, device=device)


def density(v, out, workspace, d=None, stream=None):
    """ss_density: out (3 float64 on the device) <- |v|_1, |v|_2^2, phi(v)"""
    if workspace is None:
        raise TypeError("workspace must be a tensor (density_static needs none)")
    _check("ss_density", (_marshal or _native()).density(v, out, workspace, d, stream))
    return out


def density_static(v, out, d=None, stream=None):
    """ss_density_static: ss_density on the library's own fixed scratch array (allocates nothing)"""
    _check("ss_density_static", (_marshal or _native()).density(v, out, None, d, stream))
    return out


def signum_pack_ternary(g, m, beta, tau, neg, zero, d=None, stream=None):
    """ss_signum_pack_ternary: momentum update, then this worker's ternary vote"""
    _check("ss_signum_pack_ternary", (_marshal or _native()).signum_pack_ternary(g, m, beta, tau, neg, zero, d, stream))


def quorum_vote(neg, zero, quorum, voted_neg, voted_zero, d, stream=None):
    """ss_quorum_vote: the server's ternary answer from the workers' planes"""
    _check("ss_quorum_vote", (_marshal or _native()).quorum_vote(neg, zero, quorum, voted_neg, voted_zero, d, stream))


def ternary_apply(x, neg, zero, delta, d=None, stream=None):
    """ss_ternary_apply: x <- x - delta * answer"""
    _check("ss_ternary_apply", (_marshal or _native()).ternary_apply(x, neg, zero, delta, d, stream))


def signum_vote_step_ternary(g, m, beta, tau, quorum, delta, x, voted_neg, voted_zero, d=None, stream=None):
    """ss_signum_vote_step_ternary: the whole step with abstention in one call
    (borrows memory as signum_vote_step does)"""
    _check("ss_signum_vote_step_ternary", (_marshal or _native()).signum_vote_step_ternary(
        g, m, beta, tau, quorum, delta, x, voted_neg, voted_zero, d, stream))
