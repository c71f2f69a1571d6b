"""Which kernel a call goes to (host code): the test hooks do what they say, and the dispatch lines lie where both sides were measured."""
import pytest

import paper_1412_6249_amd as pa

FWD, BWD_DATA, BWD_WEIGHT = range(3)
F32, BF16 = pa.PURINE_F32, pa.PURINE_BF16
SMALL = ((2, 38, 8, 9), (42, 38, 3, 3))


def _conv(dtype, x=SMALL[0], w=SMALL[1]):
    return [pa.purine_conv_route(p, pa.conv_desc(1, w[2] // 2), x, w, dtype) for p in range(4)]


def _fc(dtype, *nck):
    return [pa.purine_fc_route(p, *nck, dtype) for p in range(3)]


@pytest.fixture
def hook():
    yield lambda v: pa.purine_debug_force_tile(v, 0)
    pa.purine_debug_force_tile(0, 0)


def test_hooks(hook):
    large = ((128, 96, 27, 27), (256, 96, 5, 5))
    assert _conv(F32) == [1, 1, 2, 2] and _fc(F32, 20, 300, 100) == [1] * 3 and _fc(BF16, 128, 9216, 4096) == [0] * 3
    assert _conv(F32, *large)[:2] == [0, 0]
    hook(-12)
    assert _conv(BF16)[:2] == [1, 1] and _conv(F32, *large)[:2] == [1, 1] and _fc(BF16, 128, 9216, 4096) == [1] * 3
    hook(-11)
    assert _conv(F32, *large) == [0, 0, 2, 2]
    hook(-13)
    assert _conv(F32) == _conv(BF16) == [0] * 4 and _fc(F32, 20, 300, 100) == [0] * 3
    hook(0)
    assert _conv(F32) == [1, 1, 2, 2]


def test_illegal_calls_have_no_route():
    assert pa.purine_conv_route(FWD, pa.conv_desc(1, 0), (1, 3, 2, 2), (4, 3, 3, 3), F32) == 0
    assert pa.purine_conv_route(4, pa.conv_desc(1, 1), *SMALL, F32) == 0 and pa.purine_fc_route(FWD, 0, 4, 4, F32) == 0
    assert pa.purine_fc_route(FWD, 4, 4, 4, pa.PURINE_I32) == 0


@pytest.mark.parametrize("dtype, n, c, k, want", [
    (F32, 20, 300, 100, 1), (F32, 1024, 32, 32, 1),
    (F32, 8192, 32, 32, 0), (F32, 65536, 32, 32, 0), (BF16, 225580, 43, 33, 0),      # a chain of n / 256 steps; split over workgroups otherwise
    (F32, 752, 53, 49, 1), (BF16, 65536, 96, 32, 1), (BF16, 262144, 512, 512, 1)])   # not split otherwise: a longer chain
def test_fully_connected_weight_gradients_of_many_images(dtype, n, c, k, want):
    assert pa.purine_fc_route(BWD_WEIGHT, n, c, k, dtype) == want
    assert pa.purine_fc_route(BWD_WEIGHT + 1, n, c, k, dtype) == want                # the bits of dw do not depend on db


@pytest.mark.parametrize("n, c, k, want", [
    (142, 30, 3186, 1), (211369, 30, 310, 1), (19, 2770, 1599, 1), (64, 333, 100, 1),
    (7405, 2645, 108, 0), (8975, 3409, 91, 0), (5368, 2700, 203, 0), (6902, 1738, 76, 0), (1027, 4042, 207, 0)])
def test_bf16_data_gradients_whose_rows_are_no_whole_packets(n, c, k, want):
    assert pa.purine_fc_route(BWD_DATA, n, c, k, BF16) == want


@pytest.mark.parametrize("n, c, hw, k, want", [
    (5, 43, 7, 18, 0), (215, 17, 19, 274, 0), (2, 55, 9, 21, 0),      # the estimate of the general kernel holds for one tap
    (36, 49, 13, 17, 2), (16, 33, 60, 60, 2)])
def test_strided_1x1_weight_gradients_of_few_channels(n, c, hw, k, want):
    assert pa.purine_conv_route(BWD_WEIGHT, pa.conv_desc(2, 0), (n, c, hw, hw), (k, c, 1, 1), F32) == want


@pytest.mark.parametrize("n, c, k, want", [(64, 1664, 64, 0), (64, 1344, 144, 0), (128, 1664, 96, 0), (20, 1000, 100, 1), (4, 957, 93, 1)])
def test_bf16_forward_rows_that_are_whole_lines_apart(n, c, k, want):
    assert pa.purine_fc_route(FWD, n, c, k, BF16) == want
