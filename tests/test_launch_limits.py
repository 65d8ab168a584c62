"""What the library launches for vectors up to the largest that the card holds, without a GPU: the
runtime's launch call is replaced by a recorder, in a process of its own.  A launch may have at
most 2^32 - 1 threads; a call that needs more has to be cut, not refused."""
import ctypes
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


class Launch(ctypes.Structure):
    _fields_ = [("grid_x", ctypes.c_uint), ("grid_y", ctypes.c_uint), ("block_x", ctypes.c_uint),
                ("reserved", ctypes.c_uint), ("first", ctypes.c_void_p), ("kernel", ctypes.c_void_p)]


class Recorder:
    """the library with recorded launches; arguments are made-up addresses far enough apart"""

    def __init__(self, shim):
        self.shim = ctypes.CDLL(shim, mode=ctypes.RTLD_GLOBAL)
        self.lib = ctypes.CDLL(os.path.join(ROOT, "paper_1802_04434_amd", "libsignsgd.so"))
        self.next = 1 << 44

    def buffer(self, nbytes):
        at = self.next
        self.next += (int(nbytes) + (1 << 30)) & ~((1 << 30) - 1)
        return at

    def table(self, addresses):
        return (ctypes.c_void_p * len(addresses))(*addresses)

    def launches(self):
        p = ctypes.POINTER(Launch)()
        n = self.shim.recorded(ctypes.byref(p))
        return [(p[i].grid_x, p[i].grid_y, p[i].block_x, p[i].first) for i in range(n)]

    def step(self, d, M, bf16, momentum, packed=False, sums=False, scratch=0, flags=0, refuse_at=-1):
        """status, launches, and the first gradient's address; the workers share one gradient"""
        words = (d + 127) // 128 * 16
        f = ctypes.c_float
        size, vp = ctypes.c_size_t, ctypes.c_void_p
        g = self.buffer(d * (2 if bf16 else 4))
        m = self.table([self.buffer(4 * d) for _ in range(M)]) if momentum else None
        x, voted = self.buffer(4 * d), self.buffer(words)
        p = self.table([self.buffer(words) for _ in range(M)]) if packed else None
        s = vp(self.buffer(d)) if sums else None
        self.shim.record_anew(refuse_at)
        if scratch:
            rc = self.lib.ss_signum_vote_step_scratch(self.table([g] * M), bf16, m, M, f(0.9), f(0.1), vp(x), vp(voted), s,
                                                      vp(self.buffer(scratch)), size(scratch), size(d), flags, None)
        else:
            rc = self.lib.ss_signum_vote_step_ex(self.table([g] * M), bf16, m, M, f(0.9), f(0.1), vp(x), vp(voted), p, s,
                                                 size(d), flags, None)
        return rc, self.launches(), g


def threads(launch):
    return launch[0] * launch[2]


# coordinates, workers, bf16, momentum, packed_out, sums; each fits a card of 288 GB with one gradient for all workers
LARGE = [((1 << 35) + 12_345, 2, 1, False, False, False), ((1 << 35) + 1, 5, 1, False, False, False),
         ((1 << 35) + 77, 16, 1, False, False, False), ((1 << 35) - 1, 9, 1, False, False, False),
         ((1 << 34) + 5, 3, 1, False, True, True), ((1 << 34) + 5, 2, 0, False, True, True),
         ((1 << 34) - 300, 2, 1, True, True, True), ((1 << 34) + 9, 2, 1, True, False, False),
         ((1 << 34) + 4097, 1, 1, False, False, False), ((1 << 33) + 8191, 7, 0, False, False, True)]


def check_large_steps(rec):
    for case in LARGE:
        rc, launches, g = rec.step(*case)
        assert rc == 0, (case, rc)
        assert launches and all(0 < threads(t) < 1 << 32 for t in launches), (case, launches)
        d, size = case[0], 2 if case[2] else 4
        # the parts' gradients begin at multiples of 16 bytes inside the buffer, in order
        starts = [t[3] - g for t in launches if g <= t[3] < g + d * size]
        assert starts[0] == 0 and starts == sorted(starts) and all(s % 16 == 0 for s in starts), case
    # lent scratch of any size, in one launch pair as far as a launch goes
    for d, M, scratch in (((1 << 34) + 9, 2, 1 << 34), ((1 << 34) + 9, 2, 128 << 20), (1 << 33, 2, 1 << 33)):
        rc, launches, _ = rec.step(d, M, 1, True, scratch=scratch)
        assert rc == 0 and len(launches) % 2 == 0 and all(0 < threads(t) < 1 << 32 for t in launches), (d, scratch)


def check_ordinary_steps(rec):
    # below the limit nothing is cut: one launch, or two where the bits go through memory
    for d, M, packed, n in (((1 << 33), 1, False, 1), ((1 << 30) + 5, 7, False, 1), ((1 << 30) + 5, 7, True, 2),
                            (272_474, 7, True, 1), (1, 64, False, 1)):
        rc, launches, g = rec.step(d, M, 0, False, packed)
        assert rc == 0 and len(launches) == n and launches[0][3] == g, (d, M, packed, launches)


def check_packed_out_without_momentum(rec):
    # one pass while the cache holds the gradients (it is 2-30 % faster there), from 2^28 bytes on two launches
    for bf16 in (0, 1):
        for M in (2, 3, 4, 8, 16, 33):
            line = -(-(1 << 28) // (M * (2 if bf16 else 4)))
            for d, n in ((1 << 20, 1), (line // 2 + 1, 1), (line - 1, 1), (line, 2), (4 * line + 5, 2)):
                rc, launches, _ = rec.step(d, M, bf16, False, packed=True)
                assert rc == 0 and len(launches) == n, (bf16, M, d, launches)


def check_refused_steps(rec):
    # more coordinates than any launch shape ever took
    for d in ((1 << 36) + 1, 1 << 40, 1 << 61):
        rc, launches, _ = rec.step(d, 1, 1, False)
        assert rc in (-5, -6) and not launches, (d, rc)
    # a refused launch ends the call, with the launches before it enqueued
    rc, launches, _ = rec.step((1 << 35) + 1, 2, 1, False, refuse_at=1)
    assert rc == -6 and len(launches) == 1


def check_other_calls(rec):
    # calls that are not cut go up to the limit of the shape that they take for the longest vectors
    f, size, vp = ctypes.c_float, ctypes.c_size_t, ctypes.c_void_p
    d = (1 << 36) - 4096                                # a quarter of a terabyte of gradients
    for bf16 in (0, 1):
        rec.shim.record_anew(-1)
        assert rec.lib.ss_signum_pack(vp(rec.buffer(4 * d)), bf16, None, f(0.9), vp(rec.buffer(d // 8)), size(d), None) == 0
        assert len(rec.launches()) == 1 and threads(rec.launches()[0]) < 1 << 32
    d = (1 << 34) - 4096
    m, words = rec.buffer(4 * d), d // 8
    rec.shim.record_anew(-1)
    assert rec.lib.ss_signum_pack(vp(rec.buffer(4 * d)), 0, vp(m), f(0.9), vp(rec.buffer(words)), size(d), None) == 0
    assert rec.lib.ss_welford_update(vp(rec.buffer(4 * d)), 0, vp(m), vp(rec.buffer(4 * d)), size(3), size(d), None) == 0
    assert rec.lib.ss_stream_copy(vp(m), vp(rec.buffer(4 * d)), size(4 * d), None) == 0
    d = (1 << 35) - 4096
    x, bits = vp(rec.buffer(4 * d)), vp(rec.buffer(d // 8))
    assert rec.lib.ss_sign_apply(x, bits, f(0.1), size(d), None) == 0
    assert rec.lib.ss_sum_apply(x, vp(rec.buffer(d)), f(0.1), size(d), None) == 0
    assert rec.lib.ss_ternary_apply(x, bits, vp(rec.buffer(d // 8)), f(0.1), size(d), None) == 0
    assert rec.lib.ss_welford_sigma(x, size(3), vp(rec.buffer(4 * d)), size(d), None) == 0
    assert rec.lib.ss_signum_pack_ternary(vp(rec.buffer(4 * d)), 0, None, f(0.9), f(0.1), bits, vp(rec.buffer(d // 8)), size(d), None) == 0
    assert len(rec.launches()) == 8 and all(0 < threads(t) < 1 << 32 for t in rec.launches())


CHECKS = {f.__name__: f for f in (check_large_steps, check_ordinary_steps, check_packed_out_without_momentum, check_refused_steps,
                                  check_other_calls)}


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    out = str(tmp_path_factory.mktemp("recorder") / "launch_recorder.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                           "-isystem", os.path.join(rocm, "include"), os.path.join(HERE, "launch_recorder.cpp"), "-o", out])
    return out


@pytest.mark.parametrize("name", sorted(CHECKS))
def test_launches(shim, name):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), shim, name], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    CHECKS[sys.argv[2]](Recorder(sys.argv[1]))
