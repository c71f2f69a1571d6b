"""Max pooling staged in LDS: whole planes per workgroup, planes cut into bands of rows (too large for LDS, or too
few to fill the chip), runs that start and end inside a packet, gradients stored from the lanes and through LDS, rows of any width,
2x2 windows straight from memory, windows at the planes' edges, infinities and NaN. Against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from synth import gen

pytestmark = pytest.mark.gpu

# N*C planes of H x W, window, stride, pad
CASES = [
    (5, 120, 131, 3, 2, 0),     # 61 KB planes: bands forward, whole planes of windows backward
    (2, 120, 131, 3, 2, 1),
    (1, 150, 149, 3, 1, 1),     # bands both ways
    (3, 97, 101, 2, 2, 0),      # few planes: bands although a plane fits
    (1, 9, 2000, 3, 2, 1),      # a handful of rows, one or two per band
    (130, 6, 700, 3, 1, 1),     # rows that need more LDS; unmasked fp32 gradient: the kernel for packets
    (130, 6, 2001, 3, 2, 1),
    (3, 4, 2100, 3, 1, 1),      # rows that need too much: the general kernels, and in fp32 the one for packets
    (1, 4, 9001, 3, 1, 1),
    (1, 5, 9001, 3, 2, 0),
    (2, 3, 9001, 2, 2, 0),
    (2061, 7, 7, 3, 2, 1),      # several planes per workgroup, the last one not full
    (2500, 3, 5, 2, 2, 0),
    (300, 6, 11, 2, 2, 0),      # 2x2 forward: the last run of a row starts earlier; rows of three outputs and of one; padding
    (700, 4, 7, 2, 2, 0),
    (700, 5, 3, 2, 2, 0),
    (60, 9, 10, 2, 2, 1),
    (21500, 28, 28, 2, 2, 0),   # an fp32 gradient of aligned rows that leaves through LDS for its size
    (700, 13, 1, 3, 1, 1),
    (4099, 1, 2, 3, 2, 1),
]


@pytest.mark.parametrize("special", [False, True], ids=["finite", "special"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_pool_tiles(case, dtype, special):
    import paper_1412_6249_amd as pa
    from gpu_util import to_dev, to_host, tdtype, pool_bwd_in_order, DEV
    NC, H, W, k, s, p = case
    rs = np.random.default_rng(list(case))
    x = np.maximum(rs.integers(-3, 4, size=(1, NC, H, W)).astype(np.float32), 0)
    if special:
        x = np.where(rs.random(x.shape) < 0.05, np.float32("nan"), x)
        x = np.where(rs.random(x.shape) < 0.05, np.float32("-inf"), x)
        x = np.where(rs.random(x.shape) < 0.02, np.float32("inf"), x)
    P, Q = (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1
    dy = rs.uniform(-1, 1, size=(1, NC, P, Q)).astype(np.float32)
    if dtype == "bf16":
        dy = gen.quantize_bf16(dy)
    # winners as the operator defines them: the first element, then every strictly larger one, in row-major order
    xp = np.zeros((NC, H + 2 * p, W + 2 * p), np.float32)
    xp[:, p:p + H, p:p + W] = x[0]
    inside = np.zeros(xp.shape[1:], bool)
    inside[p:p + H, p:p + W] = True
    at = (np.arange(H + 2 * p)[:, None] - p) * W + np.arange(W + 2 * p)[None, :] - p
    ey, earg = np.zeros((NC, P, Q), np.float32), np.full((NC, P, Q), -1, np.int32)
    for r in range(k):
        for c in range(k):
            sl = (slice(r, r + s * (P - 1) + 1, s), slice(c, c + s * (Q - 1) + 1, s))
            v = xp[:, sl[0], sl[1]]
            take = inside[sl] & ((earg < 0) | (v > ey))
            ey, earg = np.where(take, v, ey), np.where(take, at[sl], earg)
    if not special:
        oy, oarg = oracle.maxpool_fwd(x, k, s, p)
        assert np.array_equal(oarg[0], earg) and np.array_equal(oy[0].astype(np.float32), ey)

    desc = pa.pool_desc(k, s, p)
    tx, tdy = to_dev(x, dtype), to_dev(dy, dtype)
    ty = to_dev(np.full((1, NC, P, Q), 9, np.float32), dtype)
    targ = torch.full((1, NC, P, Q), -7, dtype=torch.int32, device=DEV)
    pa.purine_maxpool_fwd(desc, tx, ty, targ)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(ty)[0], ey, equal_nan=True)
    assert np.array_equal(targ.cpu().numpy()[0], earg)

    prev = gen.quantize_bf16(rs.uniform(-1, 1, size=x.shape).astype(np.float32))
    kept = np.where(ey[None] > 0, dy, np.float32(0))
    for masked in (False, True):
        for beta in (0.0, 1.0):
            tdx = to_dev(prev, dtype) if beta else to_dev(np.full(x.shape, np.nan, np.float32), dtype)
            if masked:
                pa.purine_maxpool_bwd_relu(desc, tdy, targ, ty, tdx, beta=beta)
            else:
                pa.purine_maxpool_bwd(desc, tdy, targ, tdx, beta=beta)
            torch.cuda.synchronize()
            want = pool_bwd_in_order(kept if masked else dy, earg.reshape(dy.shape), x.shape, dtype, prev=prev if beta else None)
            assert np.array_equal(to_host(tdx), want), (masked, beta)
