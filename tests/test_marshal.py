"""What the native marshalling refuses, and that it hands over what it is given: wrong
memory, dtype, layout, length or number of tensors is an error before anything is launched."""
import ctypes
import gc
import sys

import numpy as np
import pytest
import torch

import paper_1802_04434_amd as ss

DEV = "cuda"


def test_refuses_what_is_not_a_device_tensor():
    ss.load_library()
    host = torch.zeros(64)
    bits = torch.zeros(4, dtype=torch.int32)
    with pytest.raises(TypeError, match=r"g\[0\] must live in device memory"):
        ss.signum_vote_step([host], None, 0.9, 1e-4, host, bits)
    with pytest.raises(TypeError, match=r"packed\[0\] must live"):
        ss.majority_vote([bits], bits, 64)
    with pytest.raises(TypeError, match="x must live"):
        ss.sign_apply(host, bits, 1e-4)
    with pytest.raises(TypeError, match="must be a tensor"):
        ss.signum_pack(np.zeros(64, np.float32), None, 0.9, bits)
    with pytest.raises(IndexError):
        ss.signum_vote_step([], None, 0.9, 1e-4, host, bits)
    with pytest.raises(TypeError):
        ss.majority_vote(3, bits, 64)
    with pytest.raises(TypeError):
        ss.sum_apply(host, bits, 1e-4, d=6.5)
    with pytest.raises(TypeError):
        ss.density(host, host, None)


def test_a_stacked_tensor_is_one_tensor_per_worker():
    # whatever len(), g[0] and iteration answer for is a sequence of workers; a tensor's rows are
    host = torch.zeros(64)
    bits = torch.zeros(4, dtype=torch.int32)
    for g in (torch.zeros(3, 64), torch.nn.ParameterList([host, host])):
        with pytest.raises(TypeError, match=r"g\[0\] must live in device memory"):
            ss.signum_vote_step(g, None, 0.9, 1e-4, host, bits)
        with pytest.raises(TypeError, match=r"g\[0\] must live in device memory"):
            ss.signum_vote_step_ternary(g, None, 0.9, 0.1, 1, 1e-4, host, bits, bits)
    with pytest.raises(TypeError):
        ss.signum_vote_step((t for t in [host]), None, 0.9, 1e-4, host, bits)    # no length


@pytest.mark.parametrize("d", [(1 << 64) + 8, -1, -(1 << 64) + 8])
def test_a_number_of_coordinates_is_not_cut_to_64_bits(d):
    host = torch.zeros(64)
    bits = torch.zeros(4, dtype=torch.int32)
    with pytest.raises(TypeError, match="is no number of coordinates"):
        ss.signum_pack(host, None, 0.9, bits, d=d)
    with pytest.raises(TypeError, match="is no number of coordinates"):
        ss.majority_vote([bits], bits, d)
    with pytest.raises(TypeError, match="is no number of coordinates"):
        ss.signum_vote_step([host], None, 0.9, 1e-4, host, bits, d=d)


class _NullStream:
    cuda_stream = 0


def test_a_copy_takes_anything_with_an_address_and_sizes_as_ctypes_has_them():
    # nothing is copied: no bytes, or a number of them that the library refuses
    a, b = torch.zeros(64), torch.zeros(64)
    for dst, src in ((a, b), (a.untyped_storage(), b.untyped_storage())):
        ss.stream_copy(dst, src, 0, stream=_NullStream)
        ss.stream_copy(dst, src, ctypes.c_size_t(0), stream=_NullStream)
        for odd in (8, ctypes.c_uint64(8), (1 << 64) + 8):
            with pytest.raises(ss.SignSGDError) as e:
                ss.stream_copy(dst, src, odd, stream=_NullStream)
            assert e.value.status == -5
    with pytest.raises(TypeError):
        ss.stream_copy(a, b, ctypes.c_float(8), stream=_NullStream)
    with pytest.raises(TypeError):
        ss.stream_copy(a, b, 8.0, stream=_NullStream)
    with pytest.raises((AttributeError, TypeError)):
        ss.stream_copy(np.zeros(64), b, 0, stream=_NullStream)


@pytest.mark.gpu
def test_numbers_as_ctypes_has_them():
    d, f = 1000, ctypes.c_float
    g, x = torch.randn(d, device=DEV), torch.randn(d, device=DEV)
    m = [torch.zeros(d, device=DEV) for _ in range(2)]
    x2, neg, zero, v = x.clone(), *(ss.new_bits(d, DEV) for _ in range(3))
    ss.signum_vote_step([g], [m[0]], f(0.9), f(1e-4), x, v)
    ss.signum_vote_step([g], [m[1]], 0.9, 1e-4, x2, v)
    assert torch.equal(m[0], m[1]) and torch.equal(x, x2)
    ss.signum_pack_ternary(g, None, f(0), f(0.1), neg, zero)
    ss.quorum_vote([neg], [zero], ctypes.c_int(1), *(w := [ss.new_bits(d, DEV) for _ in range(2)]), d)
    assert torch.equal(w[0], neg) and torch.equal(w[1], zero)
    mean, m2 = torch.zeros(d, device=DEV), torch.zeros(d, device=DEV)
    ss.welford_update(g, mean, m2, ctypes.c_uint64(1))
    assert torch.equal(mean, g)


@pytest.mark.gpu
def test_stacked_tensors_give_what_lists_give():
    d, M = 1024, 3
    g, m = torch.randn(M, d, device=DEV), torch.randn(M, d, device=DEV)
    x = torch.randn(d, device=DEV)
    packed = torch.zeros(M, d // 32, dtype=torch.int32, device=DEV)
    a = [t.clone() for t in (m, x)] + [ss.new_bits(d, DEV)]
    b = [t.clone() for t in (m, x)] + [ss.new_bits(d, DEV)]
    ss.signum_vote_step(g, a[0], 0.9, 1e-4, a[1], a[2], packed)
    ss.signum_vote_step(list(g), list(b[0]), 0.9, 1e-4, b[1], b[2])
    assert all(torch.equal(s, t) for s, t in zip(a, b))
    assert torch.equal(ss.majority_vote(packed, ss.new_bits(d, DEV), d), b[2])


@pytest.mark.gpu
def test_refuses_dtype_layout_length_and_number():
    d = 1000
    f = [torch.zeros(d, device=DEV) for _ in range(3)]
    bits = [ss.new_bits(d, DEV) for _ in range(3)]
    x = torch.zeros(d, device=DEV)
    with pytest.raises(TypeError, match="dtype"):
        ss.signum_pack(f[0].half(), None, 0.9, bits[0])
    with pytest.raises(TypeError, match=r"g\[1\] has dtype"):
        ss.signum_vote_step([f[0], f[1].bfloat16()], None, 0.9, 1e-4, x, bits[0])
    with pytest.raises(TypeError, match="contiguous with at least 1000"):
        ss.signum_vote_step([torch.zeros(2 * d, device=DEV)[::2]], None, 0.9, 1e-4, x, bits[0])
    with pytest.raises(TypeError, match=r"m\[0\] must be contiguous"):
        ss.signum_vote_step([f[0]], [f[1][:d - 1]], 0.9, 1e-4, x, bits[0])
    with pytest.raises(ValueError):
        ss.signum_vote_step(f[:2], f[2:], 0.9, 1e-4, x, bits[0])
    with pytest.raises(ValueError):
        ss.quorum_vote(bits[:2], bits[2:], 1, bits[0], bits[1], d)
    with pytest.raises(TypeError, match="voted has dtype"):
        ss.majority_vote(bits[:2], x, d)
    for M in (0, 65):
        with pytest.raises(ss.SignSGDError) as e:
            ss.majority_vote([bits[0]] * M, bits[1], d)
        assert e.value.status == -2
    with pytest.raises(ss.SignSGDError) as e:
        ss.sign_apply(x[1:], bits[0], 1e-4)          # 4 bytes off a 16-byte boundary
    assert e.value.status == -3
    with pytest.raises(ss.SignSGDError) as e:
        ss.signum_vote_step([x], None, 0.9, 1e-4, x, bits[0])
    assert e.value.status == -5
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_tuples_parameters_streams_and_reference_counts():
    d = 1000
    g = tuple(torch.nn.Parameter(torch.randn(d, device=DEV)) for _ in range(3))
    x = torch.zeros(d, device=DEV)
    voted = ss.new_bits(d, DEV)
    before = [sys.getrefcount(t) for t in (*g, x, voted)]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for _ in range(50):
        assert ss.signum_vote_step(g, None, 0.9, 1.0, x, voted, stream=side) is voted
    side.synchronize()
    gc.collect()
    assert [sys.getrefcount(t) for t in (*g, x, voted)] == before
    minus = sum((t.detach() < 0).int() for t in g) >= 2
    assert torch.equal(x, torch.where(minus, 50.0, -50.0))
