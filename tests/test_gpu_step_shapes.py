"""The launch shapes of the step around the edges of their tiles, bit-exact against the oracle.
The Python calls lend scratch memory to large steps with momentum, which then run as two launches; the
one-pass kernels of that size are run through the C ABI, as a captured step runs them.
With packed_out: in one pass, and from the size rules on a pack launch over all workers, then vote and
update (256 coordinates a pack block with momentum, 512 or 1,024 without, 2,048 or 4,096 a vote block,
padding to 128; fixed adders up to 16 workers, pointer tables of 16 and 64).  In one pass: the stages of
eight workers and what they leave over, and sizes beyond the size rules; both sides of each rule are in
test_gpu_stream_shapes.py."""
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
    # one worker in the streaming shape; several workers at 2^28 bytes of gradients and momentum, where scratch is lent to
    # eight and more
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
    # stages of eight workers and what they leave over, and the streaming shapes beyond 2^28 bytes
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


@pytest.mark.parametrize("d,M,dtype,flags,sums,room", [
    ((1 << 20), 8, "bf16", 0, False, 1 << 20),                  # one slab exactly
    (3 * (1 << 20) + 8191, 5, "f32", 0, False, (1 << 20) + 16384),   # three slabs, ragged end
    ((1 << 21) + 1, 9, "f32", 1, False, (1 << 20) + 8192),      # warm-up, last slab shorter
    ((1 << 21) + 33, 7, "bf16", 2, True, (1 << 20) + 8192),     # sum update with the sums
    ((1 << 20) + 1027, 17, "f32", 0, True, 1 << 22),            # sums, sign update, one slab
    ((1 << 20) + 5, 6, "f32", 2, False, 1 << 22),
    ((1 << 28) + 1057, 2, "bf16", 2, True, 1 << 29),            # vote-and-update blocks of one row
    ((1 << 20) + 64, 4, "f32", 0, False, 1 << 19),              # too little room: one pass
])
def test_step_with_lent_scratch(ss, oracle, d, M, dtype, flags, sums, room):
    import ctypes
    L = ss.load_library()
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d + M)
    T = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = [torch.randn(d, device=DEV, generator=gen).to(T) for _ in range(M)]
    m = [torch.randn(d, device=DEV, generator=gen) * 0.3 for _ in range(M)]
    x = torch.randn(d, device=DEV, generator=gen) * 0.05
    m_np = [synth.as_numpy(t).copy() for t in m]
    x_np = synth.as_numpy(x).copy()
    nbytes = M * (room // 8)
    guard = 4096
    scratch = torch.full((nbytes + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    voted = dirty_bits(ss, d)
    s_out = torch.full((d,), 99, dtype=torch.int8, device=DEV) if sums else None
    ptrs = lambda ts: (ctypes.c_void_p * len(ts))(*[t.data_ptr() for t in ts])     # noqa: E731
    rc = L.ss_signum_vote_step_scratch(ptrs(g), int(dtype == "bf16"), ptrs(m), M, 0.9, 1e-4, x.data_ptr(), voted.data_ptr(),
                                       s_out.data_ptr() if sums else None, scratch.data_ptr(), nbytes, d, flags,
                                       ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    g_np = [synth.as_numpy(t) for t in g]
    want = oracle.signum_vote_step_ex(g_np, m_np, 0.9, 1e-4, x_np, flags)
    assert np.array_equal(bits_np(voted), want[0])
    if sums:
        assert np.array_equal(s_out.cpu().numpy(), want[-1])
    for w in range(M):
        assert_same_floats(m[w], m_np[w], "m[%d]" % w)
    assert_same_floats(x, x_np, "x")
    assert bool((scratch[nbytes:] == 0xA5).all())       # nothing beyond what was lent


def test_large_step_on_streams_and_under_capture(ss):
    # the binding lends scratch on the step's own stream; a captured step takes one pass, and both agree
    d, M = (1 << 30) // 60 + 12_345, 5
    gen = torch.Generator(device=DEV)
    gen.manual_seed(9)
    g = [torch.randn(d, device=DEV, generator=gen) for _ in range(M)]
    m0 = [torch.randn(d, device=DEV, generator=gen) * 0.3 for _ in range(M)]
    x0 = torch.randn(d, device=DEV, generator=gen) * 0.05
    assert ss.load_library().ss_step_scratch_bytes(0, 1, M, d) > 0

    def fresh():
        return [t.clone() for t in m0], x0.clone(), dirty_bits(ss, d)

    results = []
    m, x, v = fresh()
    for _ in range(2):
        ss.signum_vote_step(g, m, 0.9, 1e-4, x, v)
    results.append((m, x, v))
    side = torch.cuda.Stream()
    m, x, v = fresh()
    side.wait_stream(torch.cuda.current_stream())
    for _ in range(2):
        ss.signum_vote_step(g, m, 0.9, 1e-4, x, v, stream=side)
    side.synchronize()
    results.append((m, x, v))
    m, x, v = fresh()
    graph = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        ss.signum_vote_step(g, m, 0.9, 1e-4, x, v)
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        torch.empty(1 << 24, dtype=torch.uint8, device=DEV).fill_(255)     # the program's own memory between replays
        torch.cuda.synchronize()
    results.append((m, x, v))
    torch.cuda.synchronize()
    for m, x, v in results[1:]:
        assert torch.equal(v, results[0][2])
        assert torch.equal(x.view(torch.int32), results[0][1].view(torch.int32))
        assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(m, results[0][0]))


@pytest.mark.parametrize("M,extra,flags", [(2, 1, 0), (3, 511, 2), (4, 513, 0), (6, 63, 2),
                                                  (7, 0, 0), (8, 255, 2), (13, 129, 0), (16, 32, 2),
                                                  (33, 17, 0)])
def test_bf16_gradients_without_momentum_beyond_the_cache(ss, oracle, M, extra, flags):
    # octets of coordinates per lane, from 2^28 bytes of gradients on (a tile is 512 coordinates)
    d = ((1 << 28) // (2 * M) + 511) // 512 * 512 + extra
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M)
    g = [torch.randn(d, device=DEV, generator=gen).to(torch.bfloat16) for _ in range(M)]
    special = torch.tensor([0x0000, -0x8000, 0x0001, -0x7FFF, 0x7F80, -0x0080, 0x7FC0, -0x0040], dtype=torch.int16, device=DEV)
    for t in g:                                     # zeros, subnormals, infinities and NaN of both signs
        t.view(torch.int16)[:8] = special
        t.view(torch.int16)[d - 8:] = special
    x = torch.randn(d, device=DEV, generator=gen) * 0.05
    x_np = synth.as_numpy(x).copy()
    voted = dirty_bits(ss, d)
    sums = torch.full((d,), 99, dtype=torch.int8, device=DEV)
    ss.signum_vote_step_ex(g, None, 0.9, 1e-4, x, voted, None, sums if flags else None, flags)
    want = oracle.signum_vote_step_ex([synth.as_numpy(t) for t in g], None, 0.9, 1e-4, x_np, flags)
    assert np.array_equal(bits_np(voted), want[0])
    if flags:
        assert np.array_equal(sums.cpu().numpy(), want[2])
    assert_same_floats(x, x_np, "x")


@pytest.mark.parametrize("d,M,dtype,momentum,quorum,room", [
    ((1 << 20), 8, "bf16", True, 2, 1 << 20),                       # one slab exactly
    (2 * (1 << 20) + 8191, 5, "f32", True, 1, (1 << 20) + 16384),   # two slabs, ragged end
    ((1 << 21) + 33, 9, "bf16", False, 9, (1 << 20) + 8192),        # every worker has to agree
    ((1 << 20) + 1027, 17, "f32", True, 100, 1 << 22),              # a quorum that is never met
    ((1 << 20) + 129, 64, "bf16", True, 3, 1 << 21), ((1 << 20) + 31, 33, "f32", True, 64, 1 << 21),
    ((1 << 28) + 1057, 2, "bf16", True, 2, 1 << 29),                # answer-and-update blocks of one row
    ((1 << 20) + 64, 4, "f32", True, 2, 1 << 19),                   # too little room: one pass
])
def test_ternary_step_with_lent_scratch(ss, oracle, d, M, dtype, momentum, quorum, room):
    import ctypes
    L = ss.load_library()
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d + M)
    T = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = [(torch.randn(d, device=DEV, generator=gen) * 0.3).to(T) for _ in range(M)]
    m = [torch.randn(d, device=DEV, generator=gen) * 0.2 for _ in range(M)] if momentum else None
    x = torch.randn(d, device=DEV, generator=gen) * 0.05
    m_np = [synth.as_numpy(t).copy() for t in m] if momentum else None
    x_np = synth.as_numpy(x).copy()
    nbytes = 2 * M * (room // 8)
    scratch = torch.full((nbytes + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    neg, zero = dirty_bits(ss, d), dirty_bits(ss, d)
    ptrs = lambda ts: (ctypes.c_void_p * len(ts))(*[t.data_ptr() for t in ts])     # noqa: E731
    rc = L.ss_signum_vote_step_ternary_scratch(
        ptrs(g), int(dtype == "bf16"), ptrs(m) if momentum else None, M, 0.9, 0.1, quorum, 1e-4, x.data_ptr(), neg.data_ptr(),
        zero.data_ptr(), scratch.data_ptr(), nbytes, d, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    want_neg, want_zero = oracle.signum_vote_step_ternary([synth.as_numpy(t) for t in g], m_np, 0.9, 0.1, quorum, 1e-4, x_np)
    assert np.array_equal(bits_np(neg), want_neg) and np.array_equal(bits_np(zero), want_zero)
    for w in range(M if momentum else 0):
        assert_same_floats(m[w], m_np[w], "m[%d]" % w)
    assert_same_floats(x, x_np, "x")
    assert bool((scratch[nbytes:] == 0xA5).all())


@pytest.mark.parametrize("d,M", [(d, M) for d in (1, 33, 2047, 2049, 70_001) for M in (3, 8, 9, 15, 16, 17, 33, 64)] +
                         [((1 << 22) - 1, 8), ((1 << 22) + 31, 8), ((1 << 24) - 1, 9), ((1 << 24) + 1, 17)])
def test_server_one_word_a_lane_and_four(ss, oracle, d, M):
    # sums, quorum and vote on both sides of the line between the lanes of one word and of four
    rng = np.random.default_rng(d + M)
    n = ss.packed_bytes(d) // 4
    neg = [rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32) for _ in range(M)]
    zero = [rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32) for _ in range(M)]   # both may be set
    neg_dev = [torch.from_numpy(a.view(np.int32)).to(DEV) for a in neg]
    zero_dev = [torch.from_numpy(a.view(np.int32)).to(DEV) for a in zero]
    sums = torch.full((d + 16,), 99, dtype=torch.int8, device=DEV)
    ss.vote_sum(neg_dev, sums, d)
    assert np.array_equal(sums[:d].cpu().numpy().astype(np.int32), oracle.vote_sum(neg, d))
    assert bool((sums[d:] == 99).all())
    for Q in (1, M, M + 5):
        vn, vz = dirty_bits(ss, d), dirty_bits(ss, d)
        ss.quorum_vote(neg_dev, zero_dev, Q, vn, vz, d)
        want_n, want_z = oracle.quorum_vote(neg, zero, Q, d)
        assert np.array_equal(bits_np(vn), want_n) and np.array_equal(bits_np(vz), want_z)
    voted = dirty_bits(ss, d)
    ss.majority_vote(neg_dev, voted, d)
    assert np.array_equal(bits_np(voted), oracle.majority_vote(neg, d))


def test_large_step_while_another_thread_captures(ss):
    # the scratch that the binding lends is allocated beside an open capture, which goes on unharmed
    import threading
    d, M = (1 << 30) // 60 + 77, 5
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    g = [torch.randn(d, device=DEV, generator=gen) for _ in range(M)]
    m = [torch.zeros(d, device=DEV) for _ in range(M)]
    x = torch.zeros(d, device=DEV)
    voted = dirty_bits(ss, d)
    small_x, small_v = torch.zeros(1000, device=DEV), ss.new_bits(1000, DEV)
    small_g = torch.ones(1000, device=DEV)
    own, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    failed = []

    def step():
        try:
            ss.signum_vote_step(g, m, 0.0, 1.0, x, voted, stream=other)
        except Exception as e:      # noqa: BLE001
            failed.append(e)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=own):
        ss.signum_vote_step([small_g], None, 0.0, 1.0, small_x, small_v)
        t = threading.Thread(target=step)
        t.start()
        t.join()
        ss.signum_vote_step([small_g], None, 0.0, 1.0, small_x, small_v)
    assert not failed, failed
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
    assert bool((small_x == -4).all())
    minus = sum((t < 0).int() for t in g) >= 3
    assert torch.equal(x, torch.where(minus, 1.0, -1.0))


class _Handle:
    def __init__(self, stream):
        self.cuda_stream = stream.cuda_stream


def _pointers(ts):
    import ctypes
    return (ctypes.c_void_p * len(ts))(*[t.data_ptr() for t in ts]) if ts is not None else None


def _drawn_step(d, M, dtype, momentum, scale):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d + M)
    g = [(torch.randn(d, device=DEV, generator=gen) * scale).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
         for _ in range(M)]
    m = [torch.randn(d, device=DEV, generator=gen) * 0.3 for _ in range(M)] if momentum else None
    x = torch.randn(d, device=DEV, generator=gen) * 0.05
    return g, m, x, [synth.as_numpy(t).copy() for t in m] if momentum else None, synth.as_numpy(x).copy()


def _beyond_cache(M, dtype, momentum, extra):
    """coordinates whose gradients and momentum are 2^28 bytes and a little: a step of a streaming shape"""
    size = (2 if dtype == "bf16" else 4) + (8 if momentum else 0)
    return -(-(1 << 28) // (M * size)) + extra


@pytest.mark.parametrize("M,dtype,momentum,extra,flags", [
    (2, "f32", True, 1, 3), (7, "f32", True, 2047, 0), (7, "f32", True, 0, 2), (9, "f32", True, 511, 1), (16, "f32", True, 77, 0),
    (2, "bf16", True, 2049, 0), (3, "bf16", True, 31, 2), (4, "bf16", True, 513, 1), (5, "bf16", True, 0, 0),
    (8, "bf16", True, 127, 3), (9, "bf16", True, 255, 2), (12, "bf16", True, 5, 0), (23, "bf16", True, 33, 1),
    (2, "f32", False, 2047, 2), (4, "f32", False, 1, 0), (7, "f32", False, 65, 0), (9, "f32", False, 333, 2),
])
def test_one_pass_step_beyond_the_cache(ss, oracle, M, dtype, momentum, extra, flags):
    import ctypes
    d = _beyond_cache(M, dtype, momentum, extra)
    g, m, x, m_np, x_np = _drawn_step(d, M, dtype, momentum, 1.0)
    voted = dirty_bits(ss, d)
    sums = torch.full((d,), 99, dtype=torch.int8, device=DEV)
    rc = ss.load_library().ss_signum_vote_step_ex(
        _pointers(g), int(dtype == "bf16"), _pointers(m), M, 0.9, 1e-4, x.data_ptr(), voted.data_ptr(), None,
        sums.data_ptr() if flags != 1 else None, d, flags, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    want = oracle.signum_vote_step_ex([synth.as_numpy(t) for t in g], m_np, 0.9, 1e-4, x_np, flags)
    assert np.array_equal(bits_np(voted), want[0])
    if flags != 1:
        assert np.array_equal(sums.cpu().numpy(), want[2])
    for w in range(M if momentum else 0):
        assert_same_floats(m[w], m_np[w], "m[%d]" % w)
    assert_same_floats(x, x_np, "x")


@pytest.mark.parametrize("M,dtype,momentum,extra,quorum", [
    (2, "f32", True, 1, 1), (7, "f32", True, 2047, 3), (9, "f32", True, 511, 2), (3, "bf16", True, 513, 2),
    (4, "bf16", True, 0, 1), (5, "bf16", True, 129, 2), (8, "bf16", True, 511, 9), (13, "bf16", True, 33, 2),
    (2, "bf16", False, 1023, 1), (9, "f32", False, 7, 4),
])
def test_one_pass_ternary_step_beyond_the_cache(ss, oracle, M, dtype, momentum, extra, quorum):
    import ctypes
    d = _beyond_cache(M, dtype, momentum, extra)
    g, m, x, m_np, x_np = _drawn_step(d, M, dtype, momentum, 0.3)
    neg, zero = dirty_bits(ss, d), dirty_bits(ss, d)
    rc = ss.load_library().ss_signum_vote_step_ternary(
        _pointers(g), int(dtype == "bf16"), _pointers(m), M, 0.9, 0.1, quorum, 1e-4, x.data_ptr(), neg.data_ptr(),
        zero.data_ptr(), d, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    want_neg, want_zero = oracle.signum_vote_step_ternary([synth.as_numpy(t) for t in g], m_np, 0.9, 0.1, quorum, 1e-4, x_np)
    assert np.array_equal(bits_np(neg), want_neg) and np.array_equal(bits_np(zero), want_zero)
    for w in range(M if momentum else 0):
        assert_same_floats(m[w], m_np[w], "m[%d]" % w)
    assert_same_floats(x, x_np, "x")


def _large_step(ss, extra):
    """a step for which scratch is lent; the call, binary or ternary, on fresh state and a stream, and its outputs"""
    d, M = (1 << 30) // 60 + extra, 5
    gen = torch.Generator(device=DEV)
    gen.manual_seed(extra)
    g = [torch.randn(d, device=DEV, generator=gen) for _ in range(M)]
    m0 = [torch.randn(d, device=DEV, generator=gen) * 0.3 for _ in range(M)]
    x0 = torch.randn(d, device=DEV, generator=gen) * 0.05
    assert ss.load_library().ss_step_scratch_bytes(0, 1, M, d) > 0
    assert ss.load_library().ss_ternary_scratch_bytes(0, 1, M, d) > 0

    def state():
        return [t.clone() for t in m0], x0.clone(), dirty_bits(ss, d), dirty_bits(ss, d)

    def call(state, stream, ternary):
        m, x, v, z = state
        if ternary:
            ss.signum_vote_step_ternary(g, m, 0.9, 0.1, 2, 1e-4, x, v, z, stream=stream)
        else:
            ss.signum_vote_step(g, m, 0.9, 1e-4, x, v, stream=stream)
        return [t.view(torch.int32) for t in (*m, x, v, *([z] if ternary else []))]

    return state, call


def _allocator():
    stats = torch.cuda.memory_stats()
    return {k: stats[k] for k in ("allocation.all.allocated", "reserved_bytes.all.current", "num_alloc_retries", "num_ooms")}


@pytest.mark.parametrize("ternary", [False, True])
def test_scratch_is_lent_on_torch_s_own_streams_only(ss, ternary):
    # a handle from elsewhere need not stand for one queue: there the step takes one pass and no memory
    state, call = _large_step(ss, 1001)
    pool = torch.cuda.Stream()
    external = torch.cuda.ExternalStream(pool.cuda_stream)
    states = [state() for _ in range(5)]
    torch.cuda.synchronize()
    before = _allocator()
    want = call(states[0], None, ternary)
    assert _allocator()["allocation.all.allocated"] == before["allocation.all.allocated"] + 1
    call(states[1], pool, ternary)
    pool.synchronize()
    before = _allocator()
    call(states[2], external, ternary)
    call(states[3], _Handle(pool), ternary)
    with torch.cuda.stream(external):
        call(states[4], None, ternary)
    assert _allocator() == before
    torch.cuda.synchronize()
    for m, x, v, z in states[1:]:
        got = [t.view(torch.int32) for t in (*m, x, v, *([z] if ternary else []))]
        assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("ternary", [False, True])
def test_a_step_without_room_for_scratch_leaves_the_allocator_alone(ss, ternary):
    # the program's memory is bounded to what it holds: nothing is asked for, so nothing that is cached is
    # given back, no allocation is retried and none fails
    state, call = _large_step(ss, 2002)
    states = [state() for _ in range(4)]
    torch.cuda.empty_cache()
    want = call(states[0], None, ternary)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    cached = torch.empty(300 << 20, dtype=torch.uint8, device=DEV)
    del cached
    torch.cuda.synchronize()
    total = torch.cuda.mem_get_info()[1]
    for room in (1 << 20, 1 << 29):       # less than the scratch, and more than it but little
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + room) / total)
        try:
            before = _allocator()
            got = call(states[1 if room == 1 << 20 else 2], side, ternary)
            assert _allocator() == before
        finally:
            torch.cuda.set_per_process_memory_fraction(1.0)
        side.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    before = _allocator()
    got = call(states[3], side, ternary)                # with room it is lent again
    assert _allocator()["allocation.all.allocated"] == before["allocation.all.allocated"] + 1
    side.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
