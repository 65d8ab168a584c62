"""The streaming kernels at the edges of their tiles, of the runs of tiles that a compute die takes, and on both
sides of the sizes at which a launch shape changes, bit-exact on every element: against the oracle, and for the server's calls
and the longest vectors against torch's integer and exactly rounded arithmetic on the device."""
import ctypes

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
    yield lib
    torch.cuda.empty_cache()        # the longest vectors take a hundred gigabytes


def draw(seed, d, dtype, scale):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    t = torch.randn(d, device=DEV, generator=gen).mul_(scale)
    t[::17] = 0.0
    t[5::23] = -0.0
    return t.to(torch.bfloat16 if dtype == "bf16" else torch.float32)


# A wave's tile is 256 coordinates with momentum, 512 (fp32) or 1,024 (bf16) without; eight dies take 256 tiles each in
# turn as long as there are so many, the rest goes in order.
RUNS = [(1 << 19) + e for e in (-256, -1, 0, 255, 257)] + [(1 << 20) + e for e in (-1, 0, 513)] + [(1 << 21) + e for e in (-1, 1025)] + \
       [255, 256, 511, 1025, 8 * 1024 + 3]


@pytest.mark.parametrize("momentum", [True, False])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_pack_around_runs_of_tiles(ss, oracle, dtype, momentum):
    rng = np.random.default_rng(3)
    for d in RUNS:
        g = make_grad(rng, d, dtype, scale=0.5)
        m = make_momentum(rng, d) if momentum else None
        m_dev = torch.from_numpy(m).to(DEV) if momentum else None
        packed = dirty_bits(ss, d)
        ss.signum_pack(g.to(DEV), m_dev, 0.9, packed)
        want = oracle.signum_pack(synth.as_numpy(g), m, 0.9)
        assert np.array_equal(bits_np(packed), want), d
        if momentum:
            assert_same_floats(m_dev, m, "m, d = %d" % d)


# 2^28 bytes of gradient and momentum (12 and 10 a coordinate), then 2^25 coordinates
@pytest.mark.parametrize("d,dtype", [((1 << 28) // 12, "f32"), ((1 << 28) // 12 + 1, "f32"), ((1 << 28) // 10 + 513, "bf16"),
                                     ((1 << 25) - 3, "f32"), ((1 << 25) + 300, "f32"), ((1 << 25) + 255, "bf16")])
def test_pack_on_both_sides_of_a_launch_shape(ss, oracle, d, dtype):
    g, m_dev = draw(d, d, dtype, 0.5), draw(d + 1, d, "f32", 0.3)
    m = synth.as_numpy(m_dev).copy()
    packed = dirty_bits(ss, d)
    ss.signum_pack(g, m_dev, 0.9, packed)
    want = oracle.signum_pack(synth.as_numpy(g), m, 0.9)
    assert np.array_equal(bits_np(packed), want)
    assert_same_floats(m_dev, m, "m")


# without momentum: fp32 in runs and one-wave blocks below 2^27, bf16 below 2^25, in order beyond
@pytest.mark.parametrize("d,dtype", [((1 << 27) - 513, "f32"), ((1 << 27) + 1027, "f32"), ((1 << 25) - 1, "bf16"), ((1 << 25) + 1025, "bf16")])
def test_sign_pack_on_both_sides_of_a_launch_shape(ss, oracle, d, dtype):
    g = draw(d, d, dtype, 0.5)
    packed = dirty_bits(ss, d)
    ss.signum_pack(g, None, 0.9, packed)
    assert np.array_equal(bits_np(packed), oracle.signum_pack(synth.as_numpy(g), None, 0.9))


# vote and update: a block's 2,048 (any number of workers: 4,096) coordinates, by fixed adders and by count planes, after a pack
# over lent memory; with packed_out a step of this size takes one pass.  Without momentum, for which the binding lends nothing.
@pytest.mark.parametrize("M,dtype,flags,extra", [(M, "bf16", flags, extra) for extra in (0, 1, 31, 2047, 4095)
                                                 for M, flags in ((8, 0), (16, 0), (20, 0), (9, 2), (33, 2))] +
                         [(M, "f32" if M % 2 else "bf16", 0, 2049 + M) for M in range(2, 16) if M != 8] +
                         [(33, "f32", 0, 5), (64, "bf16", 0, 8191), (3, "f32", 2, 511), (16, "f32", 2, 4097)])
def test_vote_and_update_around_a_tile(ss, oracle, M, dtype, flags, extra):
    d = (1 << 20) + extra
    g = [draw(w, d, dtype, 0.5) for w in range(M)]
    x_dev = draw(99, d, "f32", 0.05)
    x_lent, x = x_dev.clone(), synth.as_numpy(x_dev).copy()
    voted, packed = dirty_bits(ss, d), [dirty_bits(ss, d) for _ in range(M)]
    sums = torch.full((d,), 77, dtype=torch.int8, device=DEV) if flags else None
    ss.signum_vote_step_ex(g, None, 0.9, 1e-4, x_dev, voted, packed, sums, flags)
    want, want_packed, want_sums = oracle.signum_vote_step_ex([synth.as_numpy(t) for t in g], None, 0.9, 1e-4, x, flags)
    assert np.array_equal(bits_np(voted), want)
    assert all(np.array_equal(bits_np(packed[w]), want_packed[w]) for w in range(M))
    assert_same_floats(x_dev, x, "x")
    if flags:
        assert np.array_equal(sums.cpu().numpy(), want_sums)
        sums.fill_(77)
    voted.fill_(-1)
    lent = torch.empty(M * ss.packed_bytes(d), dtype=torch.uint8, device=DEV)
    table = (ctypes.c_void_p * M)(*[t.data_ptr() for t in g])
    assert ss.load_library().ss_signum_vote_step_scratch(
        table, int(dtype == "bf16"), None, M, 0.9, 1e-4, x_lent.data_ptr(), voted.data_ptr(), sums.data_ptr() if flags else None,
        lent.data_ptr(), lent.numel(), d, flags, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert np.array_equal(bits_np(voted), want)
    assert_same_floats(x_lent, x, "x over lent memory")
    if flags:
        assert np.array_equal(sums.cpu().numpy(), want_sums)


# One pass.  Runs of 64 tiles of 256 coordinates a die below 2^20 coordinates, of 256 above; the streaming shapes begin at
# 5 x 2^25 bytes of gradients and momentum, which counts twice (2^28 without momentum), one worker's at 11 x 2^23 bytes of momentum and x.
STEPS = [((1 << 17) - 1, 7, "f32", True), ((1 << 17) + 77, 16, "bf16", True), ((1 << 17) + 255, 1, "f32", True),
         ((1 << 18) + 256, 9, "f32", True), ((1 << 20) - 1, 3, "bf16", False), ((1 << 20) + 300, 6, "f32", False),
         ((5 << 25) // 84 - 1, 7, "f32", True), ((5 << 25) // 84 + 1, 7, "f32", True), ((5 << 25) // 24 + 255, 2, "f32", True),
         ((5 << 25) // 40 + 3, 4, "bf16", True), ((5 << 25) // 90 + 257, 9, "bf16", True), ((1 << 28) // 28 + 511, 7, "f32", False),
         ((1 << 28) // 8 + 300, 2, "f32", False), ((1 << 28) // 4 + 513, 2, "bf16", False), ((1 << 28) // 6 + 1, 3, "bf16", False),
         ((1 << 24) - 1, 1, "bf16", True), ((1 << 24) + 1, 1, "f32", True), ((1 << 24) + 257, 1, "bf16", False)]


@pytest.mark.parametrize("d,M,dtype,momentum", STEPS)
def test_one_pass_around_runs_and_rules(ss, oracle, d, M, dtype, momentum):
    g = [draw(d + w, d, dtype, 0.5) for w in range(M)]
    m_dev = [draw(d - w, d, "f32", 0.3) for w in range(M)] if momentum else None
    x_dev = draw(7, d, "f32", 0.05)
    m, x = [synth.as_numpy(t).copy() for t in m_dev] if momentum else None, synth.as_numpy(x_dev).copy()
    voted = dirty_bits(ss, d)
    ss.signum_vote_step(g, m_dev, 0.9, 1e-4, x_dev, voted)
    want = oracle.signum_vote_step([synth.as_numpy(t) for t in g], m, 0.9, 1e-4, x, threads=16)
    assert np.array_equal(bits_np(voted), want)
    for w in range(M if momentum else 0):
        assert_same_floats(m_dev[w], m[w], "m[%d]" % w)
    assert_same_floats(x_dev, x, "x")


# Two steps in a row, binary, with the workers' bits (the smaller ones) and with abstentions: the second reads what the first left, x in part from the
# memory-side cache.  Sizes around 16 to 92 MB written, with one worker both ends of the range in which x is kept (24 or 48 MB of x, 11 x 2^23 bytes),
# with several both sides of the line from which it is (5 x 2^25 bytes of gradients and momentum, 2^28 without).
MOST = 11 << 23
KEPT = [((1 << 24) // 32 - 1, 7, "f32", True), ((1 << 24) // 32 + 1, 7, "f32", True), (MOST // 32 - 1, 7, "f32", True), (MOST // 32, 7, "f32", True),
        ((3 << 23) // 36 + 1, 8, "bf16", True), (MOST // 36 - 255, 8, "bf16", True), (MOST // 36 + 1, 8, "f32", True),
        ((1 << 25) // 52 + 1, 12, "f32", True), ((1 << 25) // 52 - 300, 12, "bf16", True), (MOST // 40 - 1, 9, "f32", True), (MOST // 12 + 257, 2, "bf16", True),
        ((25 << 20) // 28 - 1, 3, "f32", True), ((25 << 20) // 28 + 33, 3, "f32", True), ((25 << 20) // 28 - 257, 4, "bf16", True), (10_007, 2, "f32", True),
        ((3 << 23) // 8 + 1, 1, "f32", True), ((3 << 24) // 8 - 1, 1, "bf16", True), (MOST // 8 - 1, 1, "bf16", True), (MOST // 8 + 300, 2, "f32", True), (MOST // 8 + 1, 1, "f32", True), (MOST // 4 - 1, 1, "f32", False),
        ((1 << 24) // 4 + 1, 3, "f32", False), ((1 << 28) // 28 + 257, 7, "f32", False), ((1 << 28) // 64 + 1, 16, "f32", False), (MOST // 4 - 513, 4, "f32", False),
        (MOST // 4 + 1, 4, "bf16", False)]


# The first 9 x 2^23 bytes of x are kept and the rest is not (without momentum up to eight workers): the line between tiles of 256 (bf16 gradients alone
# 512) coordinates and the ragged end behind it.
X = (9 << 23) // 4
KEPT += [(MOST // 4 + 255, 1, "f32", False), (X + 3 * 256 + 77, 1, "bf16", True), (X - 1, 2, "f32", True), (X + 257, 4, "f32", False), (X + 511, 9, "bf16", False),
         (X + 512 + 33, 8, "bf16", False), ((1 << 28) // 12 + 513, 6, "bf16", False),
         ((3 << 21) - 1, 1, "f32", False), ((3 << 21) + 513, 1, "f32", False), ((6 << 21) - 257, 1, "bf16", False), ((6 << 21) + 1, 1, "bf16", False)]


@pytest.mark.parametrize("d,M,dtype,momentum", KEPT)
def test_steps_that_leave_their_lines_in_the_caches(ss, oracle, d, M, dtype, momentum):
    g = [draw(d + w, d, dtype, 0.5) for w in range(M)]
    g_host = [synth.as_numpy(t) for t in g]
    m0, x0 = [draw(d - w, d, "f32", 0.3) for w in range(M)] if momentum else None, draw(7, d, "f32", 0.05)
    for kind in ("step", "packed", "ternary") if d * M < 20_000_000 else ("step", "ternary") if M < 7 else ("step",):
        m_dev, x_dev = [t.clone() for t in m0] if momentum else None, x0.clone()
        m, x = [synth.as_numpy(t).copy() for t in m0] if momentum else None, synth.as_numpy(x0).copy()
        packed = [dirty_bits(ss, d) for _ in range(M)] if kind == "packed" else None
        for _ in range(2):
            voted, zero = dirty_bits(ss, d), dirty_bits(ss, d)
            if kind == "ternary":
                ss.signum_vote_step_ternary(g, m_dev, 0.9, 0.1, 2, 1e-4, x_dev, voted, zero)
                want, want_zero = oracle.signum_vote_step_ternary(g_host, m, 0.9, 0.1, 2, 1e-4, x)
                assert np.array_equal(bits_np(zero), want_zero)
            else:
                ss.signum_vote_step(g, m_dev, 0.9, 1e-4, x_dev, voted, packed)
                want, want_packed = oracle.signum_vote_step(g_host, m, 0.9, 1e-4, x, want_packed=True, threads=16)
                assert all(np.array_equal(bits_np(packed[w]), want_packed[w]) for w in range(M if packed else 0))
            assert np.array_equal(bits_np(voted), want), kind
        for w in range(M if momentum else 0):
            assert_same_floats(m_dev[w], m[w], "%s m[%d]" % (kind, w))
        assert_same_floats(x_dev, x, "%s x" % kind)


# with packed_out, on both sides of the line from which two launches pay: 2^30 bytes for three to five workers, 2^28 for six and
# seven, 2^27 for eight and more; 2^28 without momentum
@pytest.mark.parametrize("d,M,dtype,momentum", [((1 << 30) // 36 - 3, 3, "f32", True), ((1 << 30) // 36 + 3, 3, "f32", True),
                                                ((1 << 27) // 80 - 1, 8, "bf16", True), ((1 << 27) // 80 + 1, 8, "bf16", True),
                                                ((1 << 25) // 2 - 1, 2, "bf16", False), ((1 << 25) // 2 + 1, 2, "bf16", False),
                                                ((1 << 24) + 300, 2, "f32", True),
                                                ((1 << 30) // 48 + 1025, 4, "f32", True), ((1 << 30) // 50 + 31, 5, "bf16", True),
                                                ((1 << 28) // 72 - 1, 6, "f32", True), ((1 << 28) // 72 + 4095, 6, "f32", True),
                                                ((1 << 28) // 70 + 255, 7, "bf16", True), ((1 << 27) // 90 + 129, 9, "bf16", True),
                                                ((1 << 27) // 144 + (1 << 17), 12, "f32", True),
                                                ((1 << 27) // 96 - 255, 8, "f32", True), ((1 << 27) // 96 + 1, 8, "f32", True),
                                                ((1 << 28) // 4 - 1, 2, "bf16", False), ((1 << 28) // 4 + 129, 2, "bf16", False),
                                                ((1 << 28) // 28, 7, "f32", False), ((1 << 28) // 28 + 1, 7, "f32", False),
                                                ((1 << 28) // 32 - 255, 16, "bf16", False), ((1 << 20) + 4097, 33, "f32", False),
                                                ((1 << 27) + 1023, 2, "f32", False)])
def test_packed_out_on_both_sides_of_two_launches(ss, oracle, d, M, dtype, momentum):
    g = [draw(d + w, d, dtype, 0.5) for w in range(M)]
    m_dev = [draw(d - w, d, "f32", 0.3) for w in range(M)] if momentum else None
    x_dev = draw(7, d, "f32", 0.05)
    m, x = [synth.as_numpy(t).copy() for t in m_dev] if momentum else None, synth.as_numpy(x_dev).copy()
    voted, packed = dirty_bits(ss, d), [dirty_bits(ss, d) for _ in range(M)]
    ss.signum_vote_step(g, m_dev, 0.9, 1e-4, x_dev, voted, packed)
    want, want_packed = oracle.signum_vote_step([synth.as_numpy(t) for t in g], m, 0.9, 1e-4, x, want_packed=True, threads=16)
    assert np.array_equal(bits_np(voted), want)
    assert all(np.array_equal(bits_np(packed[w]), want_packed[w]) for w in range(M))
    for w in range(M if momentum else 0):
        assert_same_floats(m_dev[w], m[w], "m[%d]" % w)
    assert_same_floats(x_dev, x, "x")


# the ternary step in one pass (through the C ABI nothing is lent): both sides of the rules on size and on the workers, and a
# pack of planes around the runs of tiles
@pytest.mark.parametrize("d,M,dtype,momentum", [((1 << 24) + 257, 1, "f32", True), ((5 << 25) // 48 + 3, 4, "f32", True),
                                                ((5 << 25) // 60 + 255, 5, "f32", True), ((5 << 25) // 60 - 9, 5, "f32", True),
                                                ((5 << 25) // 60 + 1, 6, "bf16", True), ((1 << 28) // 6 + 1, 3, "bf16", False),
                                                ((1 << 28) // 8 + 511, 4, "bf16", False), ((1 << 28) // 16 + 77, 4, "f32", False),
                                                ((1 << 20) + 300, 9, "f32", True), ((1 << 17) + 5, 9, "bf16", True)])
def test_one_pass_ternary_around_rules(ss, oracle, d, M, dtype, momentum):
    g = [draw(d + w, d, dtype, 0.2) for w in range(M)]
    m_dev = [draw(d - w, d, "f32", 0.2) for w in range(M)] if momentum else None
    x_dev = draw(7, d, "f32", 0.05)
    m, x = [synth.as_numpy(t).copy() for t in m_dev] if momentum else None, synth.as_numpy(x_dev).copy()
    neg, zero = dirty_bits(ss, d), dirty_bits(ss, d)
    ss.signum_vote_step_ternary(g, m_dev, 0.9, 0.1, 2, 1e-4, x_dev, neg, zero)
    want_neg, want_zero = oracle.signum_vote_step_ternary([synth.as_numpy(t) for t in g], m, 0.9, 0.1, 2, 1e-4, x)
    assert np.array_equal(bits_np(neg), want_neg) and np.array_equal(bits_np(zero), want_zero)
    for w in range(M if momentum else 0):
        assert_same_floats(m_dev[w], m[w], "m[%d]" % w)
    assert_same_floats(x_dev, x, "x")


@pytest.mark.parametrize("d,dtype,momentum", [((1 << 19) + 257, "f32", True), ((1 << 20) - 1, "bf16", False),
                                              ((1 << 28) // 12 + 255, "f32", True), ((1 << 25) + 3, "bf16", True),
                                              ((1 << 27) - 1, "f32", False), ((1 << 27) + 513, "f32", False),
                                              ((1 << 27) + 31, "bf16", False)])
def test_ternary_pack_around_rules(ss, oracle, d, dtype, momentum):
    g = draw(d, d, dtype, 0.2)
    m_dev = draw(d + 1, d, "f32", 0.2) if momentum else None
    m = synth.as_numpy(m_dev).copy() if momentum else None
    neg, zero = dirty_bits(ss, d), dirty_bits(ss, d)
    ss.signum_pack_ternary(g, m_dev, 0.9, 0.1, neg, zero)
    want_neg, want_zero = oracle.signum_pack_ternary(synth.as_numpy(g), m, 0.9, 0.1)
    assert np.array_equal(bits_np(neg), want_neg) and np.array_equal(bits_np(zero), want_zero)
    if momentum:
        assert_same_floats(m_dev, m, "m")


# updates alone, statistics and the copy: two rows a wave below 2^23 coordinates, one above, runs of 256 and 512 tiles a die
@pytest.mark.parametrize("d", [1, 511, 513, (1 << 20) - 1, (1 << 20) + 515, (1 << 23) - 1, (1 << 23) + 257, (1 << 24) + 300])
def test_updates_and_statistics_around_rules(ss, oracle, d):
    x0, words = draw(d, d, "f32", 0.05), ss.packed_bytes(d) // 4
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d)
    neg = torch.randint(-2**31, 2**31, (words,), dtype=torch.int32, device=DEV, generator=gen)
    zero = torch.randint(-2**31, 2**31, (words,), dtype=torch.int32, device=DEV, generator=gen)
    sums = torch.randint(-64, 65, (d,), dtype=torch.int8, device=DEV, generator=gen)
    bits = [bits_np(t) for t in (neg, zero)]
    for call, want in ((lambda x: ss.sign_apply(x, neg, 1e-3), lambda x: oracle.sign_apply(x, bits[0], 1e-3)),
                       (lambda x: ss.sum_apply(x, sums, 1e-3), lambda x: oracle.sum_apply(x, sums.cpu().numpy(), 1e-3)),
                       (lambda x: ss.ternary_apply(x, neg, zero, 1e-3), lambda x: oracle.ternary_apply(x, bits[0], bits[1], 1e-3))):
        x_dev, x = x0.clone(), synth.as_numpy(x0).copy()
        call(x_dev)
        want(x)
        assert_same_floats(x_dev, x, "x")
    for dtype in ("f32", "bf16"):
        g, mean_dev, m2_dev = draw(d + 1, d, dtype, 0.5), draw(d + 2, d, "f32", 0.2), draw(d + 3, d, "f32", 0.5).square_()
        mean, m2 = synth.as_numpy(mean_dev).copy(), synth.as_numpy(m2_dev).copy()
        ss.welford_update(g, mean_dev, m2_dev, 7)
        oracle.welford_update(synth.as_numpy(g), mean, m2, 7)
        assert_same_floats(mean_dev, mean, "mean")
        assert_same_floats(m2_dev, m2, "m2")
    sigma = torch.full((d,), 9.0, device=DEV)
    ss.welford_sigma(m2_dev, 7, sigma)
    assert_same_floats(sigma, oracle.welford_sigma(m2, 7), "sigma")
    to = torch.full((d + 8,), 9.0, device=DEV)
    ss.stream_copy(to, x0, d // 4 * 16)
    assert torch.equal(to[:d // 4 * 4].view(torch.int32), x0[:d // 4 * 4].view(torch.int32)) and bool((to[d // 4 * 4:] == 9).all())


# Update after update, sigma and the densities, each reading what the one before left in the caches: an update in runs below 2^24 coordinates, m2 kept
# from 2^21 on, the mean up to 5 x 2^23, sigma up to 2^26; densities in tiles of three rows below 3 x 2^18 coordinates, eight below 2^25, six beyond, a
# row being 2,048 coordinates: one tile less than a row, one and two tiles, a round of the most blocks.
# A sum's error is at most its longest chain of additions (below 800) x 2^-53 = 9e-14.
@pytest.mark.parametrize("d", [6 * 2048 - 1, 6 * 2048 + 3, (3 << 18) - 1, (3 << 18), (1 << 21) - 1, (1 << 21) + 2047, 256 * 8 * 2048 + 5, (1 << 24) + 1,
                               (1 << 25) - 1, (1 << 25) + 6 * 2048 + 1, (5 << 23) + 257, (1 << 26) - 1, (1 << 26) + 4097])
def test_statistics_in_a_row(ss, oracle, d):
    mean_dev, m2_dev = draw(d + 2, d, "f32", 0.2), draw(d + 3, d, "f32", 0.5).square_()
    mean, m2 = synth.as_numpy(mean_dev).copy(), synth.as_numpy(m2_dev).copy()
    sigma, out, work = torch.full((d,), 9.0, device=DEV), torch.zeros(2, 4, dtype=torch.float64, device=DEV), ss.new_density_workspace(DEV)
    g = [draw(d + 1, d, "f32", 0.5), draw(d + 4, d, "bf16", 0.5)]
    for n, grad in ((7, g[0]), (8, g[1])):
        ss.welford_update(grad, mean_dev, m2_dev, n)
    ss.welford_sigma(m2_dev, 8, sigma)
    ss.density(mean_dev, out[0], work)
    ss.density(sigma, out[1], work)
    for n, grad in ((7, g[0]), (8, g[1])):
        oracle.welford_update(synth.as_numpy(grad), mean, m2, n)
    assert_same_floats(mean_dev, mean, "mean")
    assert_same_floats(m2_dev, m2, "m2")
    want = oracle.welford_sigma(m2, 8)
    assert_same_floats(sigma, want, "sigma")
    assert int(work[0]) == 0
    for got, v in zip(out[:, :3].cpu().tolist(), (mean, want)):
        assert got == pytest.approx(oracle.density(v), rel=1e-12)


# ---- the server, every coordinate against torch's own arithmetic on the device (the oracle is compared with the same calls at
# smaller sizes)

WORDS = 1 << 18         # words that are compared at a time


def random_planes(d, M, n):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d + M)
    return [[torch.randint(-2**31, 2**31, (n,), dtype=torch.int32, device=DEV, generator=gen) for _ in range(M)] for _ in range(2)]


def check_server(ss, d, M, Q):
    n = ss.packed_bytes(d) // 4
    neg, zero = random_planes(d, M, n)
    sums = torch.full((d + 16,), 99, dtype=torch.int8, device=DEV)      # no sum: |99| > M
    ss.vote_sum(neg, sums, d)
    voted, vn, vz = dirty_bits(ss, d), dirty_bits(ss, d), dirty_bits(ss, d)
    ss.majority_vote(neg, voted, d)
    ss.quorum_vote(neg, zero, Q, vn, vz, d)
    assert bool((sums[d:] == 99).all())
    sums = torch.nn.functional.pad(sums[:d], (0, 32 * n - d))
    k = torch.arange(32, dtype=torch.int32, device=DEV)
    for a in range(0, n, WORDS):
        def bits(t):
            return (t[a:a + WORDS, None] >> k) & 1

        live = torch.arange(a, min(a + WORDS, n), device=DEV)[:, None] * 32 + k < d
        minus, none, only_minus = (torch.zeros(live.shape, dtype=torch.int32, device=DEV) for _ in range(3))
        for x, z in zip(neg, zero):
            x, z = bits(x), bits(z)
            minus += x
            none += z
            only_minus += x & ~z
        assert torch.equal(sums[32 * a:32 * (a + WORDS)].view(-1, 32).int(), torch.where(live, M - 2 * minus, 0)), a
        assert torch.equal(bits(voted).bool(), (2 * minus > M) & live), a
        total = M - none - 2 * only_minus
        assert torch.equal(bits(vn).bool(), (total <= -Q) & live) and torch.equal(bits(vz).bool(), (total.abs() < Q) & live), a


# a wave's tile is 8,192 coordinates, dies take 64 (sums) or 128 tiles in turn; one word a lane below 2^22 (from nine workers
# on 3 x 2^22, votes of more than sixteen 3 x 2^21); 2^26 is where caps and orders begin to change
@pytest.mark.parametrize("M", [2, 7, 12, 16, 24])
@pytest.mark.parametrize("d", [(1 << 22) - 1, (1 << 22) + 8191, (1 << 23) + 31, (3 << 21) - 7, (3 << 21) + 7, (3 << 22) - 5, (3 << 22) + 8193,
                               (1 << 26) - 3, (1 << 26) + 129])
def test_server_around_rules(ss, M, d):
    if d > 1 << 25 and M not in (2, 16):
        M = {7: 3, 12: 11, 24: 17}[M]       # other counts of planes and batches left over
    check_server(ss, d, M, 2)


# every count of planes in lanes of four words, in runs and beyond them: one plane (a single worker), two and three with the
# caps of up to three, four and more workers, six and seven
@pytest.mark.parametrize("M,d,Q", [(1, (1 << 22) + 8193, 1), (1, (1 << 26) + 129, 1), (4, (1 << 24) + 31, 1), (4, (1 << 26) + 129, 2),
                                   (5, (1 << 26) + 8191, 3), (7, (1 << 26) + 129, 2), (33, (3 << 22) + 65, 4), (33, (1 << 26) + 1, 2),
                                   (64, (3 << 22) + 8191, 9), (64, (1 << 26) + 129, 5)])
def test_server_in_lanes_of_four_words(ss, M, d, Q):
    check_server(ss, d, M, Q)


# The runs of 512 tiles and the rules of the larger vectors: votes of twelve workers and more and quorum votes of eight and more in runs from 2^27
# to 2^28, sums of eight and more from 2^26 to 2^28; sums four a batch from 2^24 on, quorum votes of up to seven from 5 x 2^22.  The
# first and the last coordinates, where the runs begin and end, and what does not fill a round of them.
@pytest.mark.parametrize("M,d", [(5, (5 << 22) - 1), (6, (5 << 22) + 33), (7, (1 << 24) - 129), (9, (1 << 24) + 1), (13, (1 << 24) + 8193), (33, (1 << 24) + 31),
                                 (9, (1 << 26) + 8191), (5, (1 << 27) - 1), (13, (1 << 27) + 4097), (20, (1 << 27) - 33), (17, (1 << 27) + 8193),
                                 (8, (1 << 27) + 1), (12, (1 << 28) - 31), (17, (1 << 28) - 8193), (9, (1 << 28) + 129), (12, (1 << 28) + 1)])
def test_server_in_long_runs(ss, M, d):
    check_server(ss, d, M, 2)


# ---- the longest vectors: shapes that only they take, the reference in chunks on the device

CHUNK = 1 << 28
LONGEST = (1 << 33) + 1283      # from 2^33 on two rows (the pack: four) a wave


def long_floats(d, seed, scale):
    t = torch.empty(d, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    for a in range(0, d, CHUNK):
        t[a:a + CHUNK].normal_(0, scale, generator=gen)
    return t


def long_words(d, seed):
    n = (d + 127) // 128 * 4
    t = torch.empty(n, dtype=torch.int32, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    for a in range(0, n, CHUNK):
        t[a:a + CHUNK].random_(-2**31, 2**31, generator=gen)
    return t


def bits_of(words, a, n):
    """the bits of coordinates a to a + n as booleans; a is a multiple of 32"""
    k = torch.arange(32, dtype=torch.int32, device=DEV)
    return ((words[a // 32:(a + n + 31) // 32, None] >> k) & 1).view(-1)[:n].bool()


# runs of tiles with 32-bit offsets up to 2^34 coordinates, 64-bit ones beyond
@pytest.mark.parametrize("d", [(1 << 34) - 33, (1 << 34) + 8193])
def test_vote_over_the_longest_vectors(ss, d):
    a, b, c = (long_words(d, seed) for seed in range(3))
    voted = dirty_bits(ss, d)
    for workers, vote in (([a], lambda x: x[0]), ([a, b], lambda x: x[0] & x[1]),
                          ([a, b, c], lambda x: (x[0] & x[1]) | (x[2] & (x[0] ^ x[1])))):
        voted.fill_(-1)
        ss.majority_vote(workers, voted, d)
        full = d // 32
        for lo in range(0, full, CHUNK):
            hi = min(lo + CHUNK, full)
            assert torch.equal(voted[lo:hi], vote([t[lo:hi] for t in workers])), (len(workers), lo)
        rest = vote([t[full:] for t in workers]).cpu()
        rest[0] &= (1 << d % 32) - 1
        rest[1:] = 0
        assert torch.equal(voted[full:].cpu(), rest)


def test_sign_pack_of_the_longest_vectors(ss):
    d = LONGEST
    g = long_floats(d, 5, 1.0)
    packed = dirty_bits(ss, d)
    ss.signum_pack(g, None, 0.9, packed)
    for a in range(0, d, CHUNK):
        n = min(CHUNK, d - a)
        assert torch.equal(bits_of(packed, a, n), g[a:a + n] < 0), a
    assert packed[d // 32].item() >> d % 32 == 0 and bool((packed[d // 32 + 1:] == 0).all())


def test_updates_and_sigma_of_the_longest_vectors(ss):
    d = LONGEST
    x, delta = torch.zeros(d, device=DEV), 0.25                   # multiples of a quarter: every sum is exact
    neg, zero = long_words(d, 1), long_words(d, 2)
    ss.sign_apply(x, neg, delta)
    ss.ternary_apply(x, neg, zero, 4 * delta)
    sums = torch.empty(d, dtype=torch.int8, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    for a in range(0, d, CHUNK):
        sums[a:a + CHUNK].random_(-64, 65, generator=gen)
    ss.sum_apply(x, sums, 16 * delta)
    for a in range(0, d, CHUNK):
        n = min(CHUNK, d - a)
        s = 1.0 - 2.0 * bits_of(neg, a, n).float()
        want = -delta * s - 4 * delta * torch.where(bits_of(zero, a, n), 0.0, s) - 16 * delta * sums[a:a + n].float()
        assert torch.equal(x[a:a + n], want), a
    del sums, neg, zero
    for a in range(0, d, CHUNK):                                  # squares, so that the root is exact
        x[a:a + CHUNK].random_(0, 4096, generator=gen).square_()
    sigma = torch.full((d,), 9.0, device=DEV)
    ss.welford_sigma(x, 1, sigma)
    for a in range(0, d, CHUNK):
        assert torch.equal(sigma[a:a + CHUNK].square(), x[a:a + CHUNK]) and bool((sigma[a:a + CHUNK] >= 0).all()), a


# the binary step runs part by part, the ternary one in two rows a wave; with momentum halved into zeros every value is exact
@pytest.mark.parametrize("M,dtype,momentum", [(2, "f32", False), (2, "bf16", False), (1, "f32", True), (1, "bf16", True)])
def test_steps_over_the_longest_vectors(ss, M, dtype, momentum):
    d, delta, tau, quorum = LONGEST, 0.25, 0.5, M
    g = []
    for w in range(M):
        t = torch.empty(d, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device=DEV)
        gen = torch.Generator(device=DEV)
        gen.manual_seed(w)
        for a in range(0, d, CHUNK):
            t[a:a + CHUNK].normal_(0, 1, generator=gen)
        g.append(t)
    m = [torch.zeros(d, device=DEV) for _ in range(M)] if momentum else None
    x, neg, zero = torch.zeros(d, device=DEV), dirty_bits(ss, d), dirty_bits(ss, d)

    def chunks():
        for a in range(0, d, CHUNK):
            n = min(CHUNK, d - a)
            v = [t[a:a + n].float() * (0.5 if momentum else 1.0) for t in g]
            if momentum:
                assert torch.equal(m[0][a:a + n], v[0]), a
                m[0][a:a + n] = 0
            yield a, n, v

    ss.signum_vote_step(g, m, 0.5, delta, x, neg)
    for a, n, v in chunks():
        minus = sum((t < 0).to(torch.int8) for t in v) >= M // 2 + 1
        assert torch.equal(bits_of(neg, a, n), minus) and torch.equal(x[a:a + n], torch.where(minus, delta, -delta)), a
        x[a:a + n] = 0
    neg.fill_(-1)
    ss.signum_vote_step_ternary(g, m, 0.5, tau, quorum, delta, x, neg, zero)
    for a, n, v in chunks():
        total = sum(torch.where(t.abs() < tau, 0, torch.where(t < 0, -1, 1)).to(torch.int8) for t in v)
        minus, none = total <= -quorum, total.abs() < quorum
        assert torch.equal(bits_of(neg, a, n), minus) and torch.equal(bits_of(zero, a, n), none), a
        assert torch.equal(x[a:a + n], torch.where(none, 0.0, torch.where(minus, delta, -delta))), a
    for t in (neg, zero):
        assert t[d // 32].item() >> d % 32 == 0 and bool((t[d // 32 + 1:] == 0).all())
