"""The fp32 kernel that splits a patch in LDS, its last tiles summed by several workgroups (a ragged last part among
them) and joined by a second launch, also behind whole rounds of 256 tiles that are not shared: every form and epilogue
against float64 sums, infinities and NaN, and the same bits from run to run. The parts' sums are added in a fixed order,
one rounding more per part than the whole sum."""
import numpy as np
import pytest

import oracle
from test_gpu_packets import _inputs, _run

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad
CASES = [(5, 96, 13, 13, 97, 3, 3, 1, 1), (2, 233, 9, 11, 45, 3, 3, 1, 1), (3, 40, 29, 31, 70, 5, 5, 1, 2), (4, 33, 27, 29, 96, 3, 3, 2, 1),
         (1, 130, 5, 23, 64, 1, 5, 1, (0, 2)), (60, 17, 4, 3, 33, 3, 3, 1, 1),
         (98, 40, 28, 28, 40, 3, 3, 1, 1), (92, 20, 56, 55, 36, 3, 3, 2, 1)]     # 256 whole tiles and a tail


def _cut(groups, parts):
    """Whether `parts` workgroups can share that many groups of 16 channels, none of them empty."""
    return parts <= groups and -(-groups // -(-groups // parts)) == parts


def _passes(case, parts):
    """The passes whose tail tiles are shared (forward: unit stride only)."""
    return [w for w, ch in ((0, case[1]), (1, case[4])) if _cut(-(-ch // 16), parts) and not (w == 0 and case[7] != 1)]


def _rel(case):
    """Half of what an fp32 chain of the longer of the two sums rounds, 2.7e-8 * sqrt(products) (the six products measured a third
    of it), and two roundings at the end."""
    return min(6e-7, 1.35e-8 * np.sqrt(max(case[1], case[4]) * case[5] * case[6]) + 6e-8)


RUNS = [(c, n) for c in CASES for n in (2, 3, 5) if _passes(c, n)]


@pytest.mark.parametrize("case, parts", RUNS, ids=["x".join(map(str, c)) + "-%d" % n for c, n in RUNS])
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
    large = case[0] * case[2] * case[3] > 30000
    if (case[0] in (3, 5) and parts < 4) or large:
        # the parts' sums outgrow what the general kernel's filter copy takes
        assert all(need[w] > whole[w] for w in _passes(case, parts) if large or w == 1)
    y = oracle.conv_fwd(x, w, stride, pad)
    dx = oracle.conv_bwd_data(dy, w, x.shape, stride, pad)
    want = [np.maximum(y + b.reshape(1, -1, 1, 1), 0), y, dx, dx + prev, dx * (act > 0)]
    for g, a, o, name in zip(got, again, want, ("relu(y + b)", "y", "dx", "dx + prev", "dx masked")):
        assert rel_l2(g, o) <= _rel(case), name
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
