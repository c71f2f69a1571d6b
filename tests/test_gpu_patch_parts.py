"""The fp32 kernel that splits a patch in LDS, its last tiles summed by several workgroups (a ragged last part among
them) and joined by a second launch: every form and epilogue against float64 sums, infinities and NaN, and the same
bits from run to run. The parts' sums are added in a fixed order, one rounding more per part than the whole sum."""
import numpy as np
import pytest

import oracle
from test_gpu_packets import _inputs, _run

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad
CASES = [(5, 96, 13, 13, 97, 3, 3, 1, 1), (2, 233, 9, 11, 45, 3, 3, 1, 1), (3, 40, 29, 31, 70, 5, 5, 1, 2), (4, 33, 27, 29, 96, 3, 3, 2, 1),
         (1, 130, 5, 23, 64, 1, 5, 1, (0, 2)), (60, 17, 4, 3, 33, 3, 3, 1, 1)]


@pytest.mark.parametrize("parts", [2, 3, 5])
@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_parts(case, parts):
    import paper_1412_6249_amd as pa
    from gpu_util import rel_l2
    x, w, b, dy, act, prev = _inputs(case)
    stride, pad = case[7], case[8]
    pa.purine_debug_force_tile(-6, 0)
    try:
        _, whole = _run(pa, case, x, w, b, dy, act, prev)
        pa.purine_debug_force_tile(-6, parts)
        got, need = _run(pa, case, x, w, b, dy, act, prev)
        again, _ = _run(pa, case, x, w, b, dy, act, prev)
    finally:
        pa.purine_debug_force_tile(0, 0)
    if case[0] in (3, 5) and parts < 4:
        assert need[1] > whole[1]                    # the parts' sums outgrow what the general kernel's filter copy takes
    y = oracle.conv_fwd(x, w, stride, pad)
    dx = oracle.conv_bwd_data(dy, w, x.shape, stride, pad)
    want = [np.maximum(y + b.reshape(1, -1, 1, 1), 0), y, dx, dx + prev, dx * (act > 0)]
    for g, a, o, name in zip(got, again, want, ("relu(y + b)", "y", "dx", "dx + prev", "dx masked")):
        assert rel_l2(g, o) <= 6e-7, name            # half of what an fp32 chain of 1200 products rounds (2.7e-8 * sqrt(1200))
        assert np.array_equal(g, a), name


def test_parts_special_values():
    import paper_1412_6249_amd as pa
    case = CASES[0]
    x, w, b, dy, act, prev = _inputs(case)
    x[0, 3, 4, 5], x[1, 90, 0, 0], x[2, 50, 12, 12] = np.inf, np.nan, -np.inf
    dy[4, 96, 3, 3], dy[3, 0, 7, 7] = np.nan, np.inf
    w[5, 95, 1, 1] = np.float32(2.0 ** 115)
    pa.purine_debug_force_tile(-6, 3)
    try:
        got, _ = _run(pa, case, x, w, b, dy, act, prev)
        pa.purine_debug_force_tile(0, -1)            # the general fp32 kernels
        ref, _ = _run(pa, case, x, w, b, dy, act, prev)
    finally:
        pa.purine_debug_force_tile(0, 0)
    for g, r in list(zip(got, ref))[1:3]:            # y, dx
        assert np.array_equal(np.isnan(g), np.isnan(r)) and np.array_equal(np.isinf(g), np.isinf(r))
        ok = np.isfinite(r)
        assert np.all(np.abs(g[ok].astype(np.float64) - r[ok]) <= 1e-4 * np.maximum(np.abs(r[ok]), 1.0))
