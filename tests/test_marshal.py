"""The native argument marshalling: what it hands back to the general path (None), which then raises as it always did."""
import numpy as np
import pytest
import torch


def test_hands_back_what_is_not_a_plain_gpu_tensor():
    import paper_1412_6249_amd as pa
    from paper_1412_6249_amd import _marshal
    x, y = torch.zeros(1, 4, 4, 4), torch.zeros(1, 4, 4, 4)
    raw = pa.raw_desc(0, pa.PURINE_F32, (1, 4, 4, 4))
    for a, b, s in ((x, y, 0), (raw, raw, 0), (None, y, 0), (object(), y, 0), (x, np.zeros(4), 0), (x, y, "stream")):
        assert _marshal.purine_relu_fwd(a, b, s) is None
    assert _marshal.purine_relu_fwd(x, y) is None and _marshal.purine_relu_fwd(x, y, 0, 0) is None
    assert _marshal.purine_conv_fwd(object(), x, x, y, None, 0) is None
    with pytest.raises(ValueError):
        pa.purine_relu_fwd(x, y, stream=0)
    with pytest.raises(pa.PurineError) as e:
        pa.purine_relu_fwd(raw, raw, stream=0)
    assert e.value.status == -1
    with pytest.raises(AttributeError):
        pa.purine_relu_fwd(None, y, stream=0)


def test_has_no_thread_local_storage():
    """A module with a TLS segment (program header type 7), loaded last, slows the thread_locals of every library loaded before."""
    import struct
    from paper_1412_6249_amd import _marshal
    data = open(_marshal.__file__, "rb").read()
    assert data[:6] == b"\x7fELF\x02\x01"
    at, = struct.unpack_from("<Q", data, 32)
    size, count = struct.unpack_from("<HH", data, 54)
    assert 7 not in [struct.unpack_from("<I", data, at + i * size)[0] for i in range(count)]


def test_descriptors_are_of_their_type_not_of_their_size():
    import ctypes
    import paper_1412_6249_amd as pa
    from paper_1412_6249_amd import _marshal

    class Derived(pa.purine_conv_desc):
        pass

    for good in (pa.conv_desc(1, 1), Derived(1, 1, 0, 0)):
        assert _marshal.takes_descriptor(good, 0) and not _marshal.takes_descriptor(good, 1)
    assert _marshal.takes_descriptor(pa.pool_desc(2, 2), 1) and not _marshal.takes_descriptor(pa.pool_desc(2, 2), 0)
    for size, which, call in ((16, 0, lambda d: pa.purine_conv_fwd(d, pa.raw_desc(0, 0, (1, 4, 4, 4)), pa.raw_desc(0, 0, (1, 4, 1, 1)), pa.raw_desc(0, 0, (1, 1, 4, 4)), stream=0)),
                              (12, 1, lambda d: pa.purine_maxpool_fwd(d, pa.raw_desc(0, 0, (1, 4, 4, 4)), pa.raw_desc(0, 0, (1, 4, 2, 2)), pa.raw_desc(0, 2, (1, 4, 2, 2)), stream=0))):
        for bad in (bytes(size), bytearray(size), np.zeros(size // 4, np.int32), (ctypes.c_int32 * (size // 4))()):
            assert not _marshal.takes_descriptor(bad, which)
            with pytest.raises((TypeError, ctypes.ArgumentError)):
                call(bad)


@pytest.mark.gpu
def test_same_call_and_same_refusals_as_the_general_path():
    import ctypes
    import paper_1412_6249_amd as pa
    from paper_1412_6249_amd import _marshal
    dev = "cuda:0"
    big = torch.randn(3, 24, 5, 6, device=dev)
    x, side = big[:, 8:16], torch.cuda.Stream()
    y = torch.zeros(3, 8, 5, 6, device=dev)
    pa.purine_relu_fwd(x, y)
    assert torch.equal(y, x.clamp(min=0))
    y.zero_()
    torch.cuda.synchronize()
    for stream in (side, side.cuda_stream):
        pa.purine_relu_fwd(x, y, stream=stream)
        side.synchronize()
        assert torch.equal(y, x.clamp(min=0))
        y.zero_()
        torch.cuda.synchronize()
    with torch.cuda.stream(side):                       # the current stream
        pa.purine_relu_fwd(x, y)
        side.synchronize()
    assert torch.equal(y, x.clamp(min=0))
    # a descriptor beside a tensor; errors of the entry point; forms that are refused before it
    pa.purine_relu_fwd(pa.tensor_desc(x), y)
    with pytest.raises(pa.PurineError) as e:
        pa.purine_relu_fwd(x, y[:, :4].contiguous())
    assert e.value.status == -2
    for bad in (x.transpose(2, 3), big[:, ::2], x.double(), torch.zeros(1, 1, 1, 1, 1, device=dev)):
        assert _marshal.purine_relu_fwd(bad, y, None) is None
        with pytest.raises((ValueError, TypeError)):
            pa.purine_relu_fwd(bad, y)
    # objects that only have a descriptor's size
    w1, y1, arg = torch.randn(8, 24, 1, 1, device=dev), torch.empty(3, 8, 5, 6, device=dev), torch.empty(3, 24, 2, 3, dtype=torch.int32, device=dev)
    for bad in (bytes(16), np.ones(4, np.int32), (ctypes.c_int32 * 4)(1, 1, 0, 0)):
        assert _marshal.purine_conv_fwd(bad, big, w1, y1, None, None) is None
        with pytest.raises((TypeError, ctypes.ArgumentError)):
            pa.purine_conv_fwd(bad, big, w1, y1)
    for bad in (bytes(12), np.array([2, 2, 0], np.int32)):
        assert _marshal.purine_maxpool_fwd(bad, big, torch.empty(3, 24, 2, 3, device=dev), arg, None) is None
    desc = pa.conv_desc(1, 1)
    w, out = torch.randn(8, 24, 3, 3, device=dev), torch.empty(3, 8, 5, 6, device=dev)
    with pytest.raises(pa.PurineError) as e:
        pa.purine_conv_fwd(desc, big, w, out)            # no scratch
    assert e.value.status == -5
    with pytest.raises(ctypes.ArgumentError):
        pa.purine_conv_fwd(pa.pool_desc(2, 2), big, w, out)
