"""The launch shapes of the step around the edges of their tiles, bit-exact against the oracle.
With packed_out from about 2^20 coordinates on: a pack launch over all workers, then vote and
update (256 coordinates a pack block with momentum, 1,024 without, 1,024 to 4,096 a vote block,
padding to 128; fixed adders up to 16 workers, pointer tables of 16 and 64).  In one pass: the
stages of eight workers and what they leave over, and both sides of the size rules."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_parity import DEV, assert_same_floats, bits_np, dirty_bits, make_grad, make_momentum

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ss():
    import paper_1802_04434_amd as lib
    lib.load_library()
    return lib


@pytest.mark.parametrize("d,M,dtype,momentum", [
    ((1 << 20), 8, "f32", True), ((1 << 20) + 1, 9, "bf16", True), ((1 << 20) + 255, 16, "f32", False),
    ((1 << 20) + 1023, 16, "bf16", False), ((1 << 20) + 4095, 17, "f32", True), ((1 << 20) + 129, 64, "bf16", False),
    ((1 << 21) + 33, 5, "f32", True), ((1 << 23) + 4097, 2, "bf16", True), ((1 << 23) + 31, 3, "f32", False),
    ((1 << 28) + 1057, 2, "bf16", False),
])
def test_step_with_packed_out(ss, oracle, d, M, dtype, momentum):
    rng = np.random.default_rng(d + M)
    if d <= 1 << 24:
        g = [make_grad(rng, d, dtype, scale=0.5) for _ in range(M)]
        g_dev = [t.to(DEV) for t in g]
    else:
        gen = torch.Generator(device=DEV)
        gen.manual_seed(M)
        g_dev = [torch.randn(d, device=DEV, generator=gen).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
                 for _ in range(M)]
        g = [t.cpu() for t in g_dev]
    m = [make_momentum(rng, d) for _ in range(M)] if momentum else None
    x = (rng.standard_normal(d, dtype=np.float32) * np.float32(0.05))
    m_dev = [torch.from_numpy(a).to(DEV) for a in m] if momentum else None
    x_dev = torch.from_numpy(x).to(DEV)
    voted = dirty_bits(ss, d)
    packed = [dirty_bits(ss, d) for _ in range(M)]
    ss.signum_vote_step(g_dev, m_dev, 0.9, 1e-4, x_dev, voted, packed)
    want_voted, want_packed = oracle.signum_vote_step([synth.as_numpy(t) for t in g], m, 0.9, 1e-4, x,
                                                      want_packed=True, threads=16)
    assert np.array_equal(bits_np(voted), want_voted)
    for w in range(M):
        assert np.array_equal(bits_np(packed[w]), want_packed[w]), w
        if momentum:
            assert_same_floats(m_dev[w], m[w], "m[%d]" % w)
    assert_same_floats(x_dev, x, "x")


@pytest.mark.parametrize("d", [255, 256 * 5 + 1, 70_001])
@pytest.mark.parametrize("M,momentum", [(9, True), (10, False), (11, True), (12, True), (13, False), (14, True), (15, True),
                                        (16, False), (23, True), (33, True)])
def test_small_step_with_workers_left_over(ss, oracle, d, M, momentum):
    # a stage takes eight workers; the 1 .. 7 left over are one stage of that size
    rng = np.random.default_rng(d + M)
    dtype = "bf16" if M % 3 == 0 else "f32"
    g = [make_grad(rng, d, dtype, scale=0.5) for _ in range(M)]
    m = [make_momentum(rng, d) for _ in range(M)] if momentum else None
    x = (rng.standard_normal(d) * 0.05).astype(np.float32)
    m_dev = [torch.from_numpy(a).to(DEV) for a in m] if momentum else None
    x_dev = torch.from_numpy(x).to(DEV)
    voted = dirty_bits(ss, d)
    ss.signum_vote_step([t.to(DEV) for t in g], m_dev, 0.9, 1e-4, x_dev, voted)
    want_voted = oracle.signum_vote_step([synth.as_numpy(t) for t in g], m, 0.9, 1e-4, x)
    assert np.array_equal(bits_np(voted), want_voted)
    for w in range(M if momentum else 0):
        assert_same_floats(m_dev[w], m[w], "m[%d]" % w)
    assert_same_floats(x_dev, x, "x")


@pytest.mark.parametrize("d,M,dtype,momentum", [
    ((1 << 25) + 255, 1, "f32", True), ((1 << 25) + 256, 1, "bf16", False),
    ((1 << 28) // 84 - 5, 7, "f32", True), ((1 << 28) // 80 + 77, 8, "bf16", True),
])
def test_step_on_both_sides_of_a_launch_shape(ss, oracle, d, M, dtype, momentum):
    # one worker from 2^25 coordinates on; several workers at 2^28 bytes of gradients and momentum
    rng = np.random.default_rng(d)
    g = [make_grad(rng, d, dtype, scale=0.5) for _ in range(M)]
    m = [make_momentum(rng, d) for _ in range(M)] if momentum else None
    x = (rng.standard_normal(d, dtype=np.float32) * np.float32(0.05))
    m_dev = [torch.from_numpy(a).to(DEV) for a in m] if momentum else None
    x_dev = torch.from_numpy(x).to(DEV)
    voted = dirty_bits(ss, d)
    ss.signum_vote_step([t.to(DEV) for t in g], m_dev, 0.9, 1e-4, x_dev, voted)
    want_voted = oracle.signum_vote_step([synth.as_numpy(t) for t in g], m, 0.9, 1e-4, x, threads=16)
    assert np.array_equal(bits_np(voted), want_voted)
    for w in range(M if momentum else 0):
        assert_same_floats(m_dev[w], m[w], "m[%d]" % w)
    assert_same_floats(x_dev, x, "x")


@pytest.mark.parametrize("d,M,dtype,momentum", [
    (1, 9, "f32", True), (255, 8, "bf16", True), (257, 15, "f32", False), (70_001, 16, "bf16", True), (70_001, 23, "f32", False),
    ((1 << 28) // 28 + 511, 7, "f32", False), ((1 << 28) // 32 + 1, 16, "bf16", False), ((1 << 28) // 24 - 300, 2, "f32", True),
])
def test_ternary_step(ss, oracle, d, M, dtype, momentum):
    # stages of eight workers and what they leave over, and both sides of the 2^28-byte rule
    rng = np.random.default_rng(d + M)
    g = [make_grad(rng, d, dtype, scale=0.2) for _ in range(M)]
    m = [make_momentum(rng, d) for _ in range(M)] if momentum else None
    x = (rng.standard_normal(d) * 0.05).astype(np.float32)
    m_dev = [torch.from_numpy(a).to(DEV) for a in m] if momentum else None
    x_dev = torch.from_numpy(x).to(DEV)
    neg, zero = dirty_bits(ss, d), dirty_bits(ss, d)
    ss.signum_vote_step_ternary([t.to(DEV) for t in g], m_dev, 0.9, 0.1, 2, 1e-4, x_dev, neg, zero)
    want_neg, want_zero = oracle.signum_vote_step_ternary([synth.as_numpy(t) for t in g], m, 0.9, 0.1, 2, 1e-4, x)
    assert np.array_equal(bits_np(neg), want_neg) and np.array_equal(bits_np(zero), want_zero)
    for w in range(M if momentum else 0):
        assert_same_floats(m_dev[w], m[w], "m[%d]" % w)
    assert_same_floats(x_dev, x, "x")
