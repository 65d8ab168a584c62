"""Which kernel a step takes on each side of the rules on size, workers and type, without a GPU: the recorder of
test_launch_limits notes the kernel of every launch, and its name holds the launch shape."""
import ctypes
import os
import re
import subprocess
import sys

import pytest

from test_launch_limits import Launch, Recorder, shim  # noqa: F401

STREAM, KEEP, THROUGH = 2, 16, 18       # store policies: the L2 writes back, left in the memory-side cache, sent on

PARAMETERS = {"step_kernel": "MT NPTR BLOCK BW R HOLD NEAR STORE STORE_X CHUNK HAS_M",
              "step_bf16_kernel": "MT NPTR BLOCK BW HOLD STORE STORE_X",
              "ternary_step_kernel": "BW R HOLD NEAR STORE CHUNK HAS_M VOTE",
              "welford_update_kernel": "HOLD STORE_MEAN STORE_M2 CHUNK"}


class DlInfo(ctypes.Structure):
    _fields_ = [("fname", ctypes.c_char_p), ("fbase", ctypes.c_void_p), ("sname", ctypes.c_char_p), ("saddr", ctypes.c_void_p)]


def shape(symbol):
    """kernel and, of those above, the launch shape as a dict"""
    kernel = re.match(r"_ZN2ss(\d+)", symbol)
    kernel = symbol[kernel.end():kernel.end() + int(kernel.group(1))]
    values = [int(v) for v in re.findall(r"L[ijb](\d+)E", symbol)]
    names = PARAMETERS.get(kernel, "").split()
    assert not names or len(names) == len(values), symbol
    return kernel, dict(zip(names, values))


class Rules(Recorder):
    def kernels(self):
        p = ctypes.POINTER(Launch)()
        n = self.shim.recorded(ctypes.byref(p))
        info, symbols = DlInfo(), []
        for i in range(n):
            assert ctypes.CDLL(None).dladdr(ctypes.c_void_p(p[i].kernel), ctypes.byref(info)) and info.saddr == p[i].kernel
            symbols.append(info.sname.decode())
        return symbols

    def step_shapes(self, d, M, bf16, momentum, **how):
        rc, _, _ = self.step(d, M, bf16, momentum, **how)
        assert rc == 0
        return [shape(s) for s in self.kernels()]

    def ternary_shapes(self, d, M, bf16, momentum):
        f, vp, words = ctypes.c_float, ctypes.c_void_p, (d + 127) // 128 * 16
        g = self.buffer(d * (2 if bf16 else 4))
        m = self.table([self.buffer(4 * d) for _ in range(M)]) if momentum else None
        self.shim.record_anew(-1)
        assert self.lib.ss_signum_vote_step_ternary(self.table([g] * M), bf16, m, M, f(0.9), f(0.1), 2, f(0.1), vp(self.buffer(4 * d)),
                                                    vp(self.buffer(words)), vp(self.buffer(words)), ctypes.c_size_t(d), None) == 0
        return [shape(s) for s in self.kernels()]


def check_ternary_steps_have_one_store_policy(rules):
    # a second policy, for tiles of x that are kept, made these kernels 1-15 % slower
    for M in (1, 2, 3, 4, 5, 7, 8, 16, 33, 64):
        for bf16 in (0, 1):
            for momentum in (True, False):
                for d in (10_007, 700_001, 2_500_003, 8_000_001, 18_000_001, 25_557_032, 60_000_001, 400_000_001):
                    (kernel, s), = rules.ternary_shapes(d, M, bf16, momentum)
                    assert kernel == "ternary_step_kernel" and s["VOTE"] and s["STORE"] in (STREAM, KEEP, THROUGH), (M, d, s)


def check_small_steps_leave_their_lines_to_the_l2(rules):
    # not to every cache: up to 35 % slower where many vectors are stepped in turn
    for M in range(2, 9):
        for bf16 in (0, 1):
            for d in (257, 10_007, 100_003, 272_474, (25 << 20) // (8 * M + 4) - 1, 400_001):
                (kernel, s), = rules.step_shapes(d, M, bf16, True)
                assert kernel == "step_kernel" and s["NEAR"] and s["STORE"] == s["STORE_X"] == STREAM, (M, bf16, d, s)


def check_lines_of_steps_with_momentum(rules):
    # bytes of gradients and momentum, which counts twice: the streaming shapes, and with packed_out the second launch
    for bf16 in (0, 1):
        for M in (2, 3, 4, 5, 7, 8, 9, 12, 16, 17, 33, 64):
            size = M * (10 if bf16 else 12)
            line = -(-(5 << 25) // size)
            (_, before), = rules.step_shapes(line - 1, M, bf16, True)
            (_, behind), = rules.step_shapes(line, M, bf16, True)
            assert before["NEAR"] and before["HOLD"] == 0 and not behind["NEAR"] and behind["HOLD"] and behind["STORE"] == THROUGH, (M, bf16)
            before, behind = rules.ternary_shapes(line - 1, M, bf16, True), rules.ternary_shapes(line, M, bf16, True)
            assert before[0][1]["NEAR"] and not behind[0][1]["NEAR"] and behind[0][1]["STORE"] == THROUGH, (M, bf16)
            if M == 2:
                continue
            line = max(-(-(1 << (27 if M >= 8 else 28 if M >= 6 else 30)) // size), 1 << 20)     # nor below 2^20 coordinates
            for d, kernels in ((line - 1, ["step_kernel"]), (line, ["pack_kernel", "vote_apply_kernel"])):
                assert [k for k, _ in rules.step_shapes(d, M, bf16, True, packed=True)] == kernels, (M, bf16, d)


def check_momentum_is_not_kept_in_the_cache(rules):
    # of what a step writes only x is ever left in the memory-side cache
    for M in (1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 33, 64):
        for bf16 in (0, 1):
            for momentum in (True, False):
                for written in (10e6, 20e6, 30e6, 50e6, 70e6, 91e6, 95e6, 300e6):
                    d = int(written) // (4 * (M + 1 if momentum else 1))
                    for kernel, s in rules.step_shapes(d, M, bf16, momentum) + rules.ternary_shapes(d, M, bf16, momentum):
                        assert s["STORE"] != KEEP or M == 1 and not momentum, (M, bf16, momentum, d, s)


def check_which_steps_keep_x(rules):
    # the streaming shapes of steps that move less than 2^31 bytes, of up to eight workers where there is no momentum
    for M in (2, 3, 4, 5, 6, 7, 8, 9, 12, 16, 17, 33, 64):
        for bf16 in (0, 1):
            for momentum in (True, False):
                size = (2 if bf16 else 4) + (8 if momentum else 0)
                line, most = -(-(5 << 25 if momentum else 1 << 28) // (M * size)), -(-(1 << 31) // (M * size + 8))
                for d, kept in ((line, True), (line + 1003, True), (most - 1, True), (most, False), (2 * most, False)):
                    for flags, sums in ((0, False), (2, False), (0, True)):
                        (_, s), = rules.step_shapes(d, M, bf16, momentum, flags=flags, sums=sums)
                        keeps = kept and not flags and not sums and (momentum or M <= 8)
                        assert (s["STORE_X"] == KEEP) == keeps and (keeps or s["STORE_X"] == s["STORE"]), (M, bf16, momentum, d, flags, sums, s)


def check_what_an_update_of_the_statistics_keeps(rules):
    # nothing below 2^21 coordinates, both below 5 x 2^23, then m2
    vp, size = ctypes.c_void_p, ctypes.c_size_t
    for bf16 in (0, 1):
        for d, mean, m2 in ((1000, STREAM, STREAM), ((1 << 21) - 1, STREAM, STREAM), (1 << 21, KEEP, KEEP), ((1 << 24) - 1, KEEP, KEEP), (1 << 24, KEEP, KEEP),
                            ((5 << 23) - 1, KEEP, KEEP), (5 << 23, THROUGH, KEEP), (400_000_001, THROUGH, KEEP)):
            rules.shim.record_anew(-1)
            assert rules.lib.ss_welford_update(vp(rules.buffer(4 * d)), bf16, vp(rules.buffer(4 * d)), vp(rules.buffer(4 * d)), size(3), size(d), None) == 0
            (kernel, s), = [shape(t) for t in rules.kernels()]
            assert kernel == "welford_update_kernel" and (s["STORE_MEAN"], s["STORE_M2"]) == (mean, m2), (bf16, d, s)
            assert (s["CHUNK"] == 9) == (d < 1 << 24)


def check_lines_of_one_worker(rules):
    # 11 x 2^23 bytes of momentum and x, where the streaming shape begins; without momentum x is kept from 24 MB (bf16 48 MB) on
    for bf16 in (0, 1):
        for momentum in (True, False):
            line, kept = -(-(11 << 23) // (8 if momentum else 4)), (6 if bf16 else 3) << 21
            for d in (1000, kept - 1, kept, (1 << 24) - 1, 1 << 24, line - 1, line, 4 * line):
                (_, s), = rules.step_shapes(d, 1, bf16, momentum)
                (_, t), = rules.ternary_shapes(d, 1, bf16, momentum)
                store = THROUGH if d >= line else KEEP if d >= kept and not momentum else STREAM
                assert s["STORE"] == t["STORE"] == store and s["NEAR"] == t["NEAR"] == (d < line), (bf16, momentum, d, s, t)
                assert s["STORE_X"] == (KEEP if d >= line else store), (bf16, momentum, d, s)


def check_every_kernel_is_reached(rules):
    # the launch shapes that the library holds are those that some call takes
    seen = set()
    f, vp, size = ctypes.c_float, ctypes.c_void_p, ctypes.c_size_t
    L = rules.lib

    def call(fn, *args):
        rules.shim.record_anew(-1)
        if fn(*args) == 0:
            seen.update(rules.kernels())

    for M in range(1, 65):
        for bf16 in (0, 1):
            for momentum in (True, False):
                worker = (2 if bf16 else 4) + (8 if momentum else 0)
                lines = [-(-b // (M * worker)) for b in (5 << 25, 1 << 27, 1 << 28, 1 << 30, 1 << 31)] + [-(-(1 << 31) // (M * worker + 8))]
                lines += [1 << 20, 1 << 24, 3 << 21, 6 << 21, -(-(11 << 23) // 4), -(-(11 << 23) // 8), 1 << 28, 1 << 33]
                for d in sorted({e for line in lines for e in (line - 1, line, 2 * line)} | {1000}):
                    for how in ({}, {"sums": True}, {"packed": True}, {"packed": True, "sums": True}):
                        if rules.step(d, M, bf16, momentum, **how)[0] == 0:
                            seen.update(rules.kernels())
                    rules.ternary_shapes(d, M, bf16, momentum)
                    seen.update(rules.kernels())
                    g, x, v, z = [rules.buffer(4 * d) for _ in range(4)]
                    m = rules.table([rules.buffer(4 * d) for _ in range(M)]) if momentum else None
                    call(L.ss_signum_vote_step_ternary_scratch, rules.table([g] * M), bf16, m, M, f(0.9), f(0.1), 2, f(0.1), vp(x), vp(v), vp(z),
                         vp(rules.buffer(1 << 40)), size(1 << 40), size(d), None)
        for d in sorted({e for p in range(20, 36) for q in (1 << p, 3 << p, 5 << p) for e in (q - 1, q)} | {1000}):
            words = (d + 127) // 128 * 16
            neg, zero = rules.table([rules.buffer(words) for _ in range(M)]), rules.table([rules.buffer(words) for _ in range(M)])
            call(L.ss_majority_vote, neg, M, vp(rules.buffer(words)), size(d), None)
            call(L.ss_vote_sum, neg, M, vp(rules.buffer(d)), size(d), None)
            call(L.ss_quorum_vote, neg, zero, M, 2, vp(rules.buffer(words)), vp(rules.buffer(words)), size(d), None)
            if M > 1:
                continue
            a, b, c, n = vp(rules.buffer(4 * d)), vp(rules.buffer(4 * d)), vp(rules.buffer(4 * d)), size(d)
            call(L.ss_sign_apply, a, b, f(0.1), n, None)
            call(L.ss_sum_apply, a, b, f(0.1), n, None)
            call(L.ss_ternary_apply, a, b, c, f(0.1), n, None)
            call(L.ss_welford_sigma, a, size(3), b, n, None)
            call(L.ss_density, a, n, b, c, None)
            call(L.ss_stream_copy, a, b, size(4 * d), None)
            for bf16 in (0, 1):
                call(L.ss_welford_update, a, bf16, b, c, size(3), n, None)
                for m in (None, c):
                    call(L.ss_signum_pack, a, bf16, m, f(0.9), b, n, None)
                    call(L.ss_signum_pack_ternary, a, bf16, m, f(0.9), f(0.1), b, vp(rules.buffer(d // 8 + 16)), n, None)
    held = subprocess.run(["nm", "-D", "--defined-only", L._name], capture_output=True, text=True, check=True).stdout
    held = {t.split()[-1] for t in held.splitlines() if t.split()[1] in "VD" and t.split()[-1].startswith("_ZN2ss")}
    assert seen <= held and held == seen, sorted(held - seen)


def check_gpu_tests_reach_both_sides(rules):
    # the lists of sizes in test_gpu_stream_shapes straddle the rules that they name
    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    import test_gpu_stream_shapes as gpu

    def parameters(test):
        return [mark.args[1] for mark in test.pytestmark if mark.name == "parametrize"][0]

    def groups(M, momentum):
        return 1 if M == 1 else 2 if not momentum or M == 2 else 3 if M < 6 else 6 if M < 8 else 8 if M < 17 else 17

    launches, steps, ternary, kept = {}, {}, {}, {}
    for d, M, dtype, momentum in parameters(gpu.test_packed_out_on_both_sides_of_two_launches):
        n = len(rules.step_shapes(d, M, int(dtype == "bf16"), momentum, packed=True))
        launches.setdefault((momentum, groups(M, momentum)), set()).add(n)
    assert all(launches[g] == {1, 2} for g in ((True, 3), (True, 6), (True, 8), (False, 2))) and launches[True, 2] == {1}, launches
    for d, M, dtype, momentum in gpu.STEPS + gpu.KEPT:
        (_, s), = rules.step_shapes(d, M, int(dtype == "bf16"), momentum)
        steps.setdefault((M > 1, momentum), set()).add((s.get("NEAR", 0), s["STORE"], s["STORE_X"]))
        if d % 256 and 4 * d > 9 << 23 and s["STORE_X"] == KEEP != s["STORE"]:
            kept.setdefault(M > 1, set()).add(d)
    near, streaming = (1, STREAM, STREAM), (0, THROUGH, KEEP)
    for group, shapes in steps.items():
        assert {near, streaming} <= shapes, (group, shapes)
    assert (1, KEEP, KEEP) in steps[False, False] and (0, THROUGH, THROUGH) in steps[True, False] and len(kept[False]) > 1 and len(kept[True]) > 1
    for d, M, dtype, momentum in parameters(gpu.test_one_pass_ternary_around_rules):
        (_, s), = rules.ternary_shapes(d, M, int(dtype == "bf16"), momentum)
        ternary.setdefault(momentum, set()).add((s["NEAR"], s["STORE"], s["HOLD"]))
    assert ternary[True] == {(1, STREAM, 0), (0, THROUGH, 11), (0, THROUGH, 12), (0, THROUGH, 13)}, ternary
    assert ternary[False] == {(0, THROUGH, 7), (0, THROUGH, 10)}, ternary


CHECKS = {f.__name__: f for f in (check_ternary_steps_have_one_store_policy, check_small_steps_leave_their_lines_to_the_l2,
                                  check_lines_of_steps_with_momentum, check_momentum_is_not_kept_in_the_cache,
                                  check_which_steps_keep_x, check_what_an_update_of_the_statistics_keeps,
                                  check_lines_of_one_worker, check_every_kernel_is_reached,
                                  check_gpu_tests_reach_both_sides)}


@pytest.mark.parametrize("name", sorted(CHECKS))
def test_rules(shim, name):  # noqa: F811
    r = subprocess.run([sys.executable, os.path.abspath(__file__), shim, name], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    CHECKS[sys.argv[2]](Rules(sys.argv[1]))
