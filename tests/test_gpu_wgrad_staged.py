"""Weight gradients whose operands are laid out inside LDS: every tile, row tiles and columns that are not full, several channel
tiles of unequal width, filter rows cut by a tile, strides, rows of no whole units of four, segments, bands (batches that are no
multiple of eight images, also ones whose rows they do not divide), planes that are no whole packets, channel-slice views, one
split (straight into dw) and many, accumulation, infinities. Against float64 sums on the CPU.

Bound: fp32 as for the other kernels on three bf16 parts (2.7e-8 * sqrt(products) is an fp32 chain's rounding, three quarters of it
and the last roundings are allowed). bf16: products are exact in fp32, so the chain's rounding is the whole error; an fp32 chain of
n products is allowed."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad
CASES = [
    (8, 3, 19, 21, 40, 7, 7, 2, 3),        # eight whole images
    (9, 3, 30, 29, 97, 11, 11, 4, 0),      # a group of one image; 363 columns over three tiles
    (3, 5, 11, 13, 33, 3, 3, 1, 1),        # bands that do not divide the rows
    (1, 20, 9, 33, 130, 3, 3, 1, 1),       # eight bands of one image
    (2, 37, 8, 7, 20, 3, 3, 2, 0),         # channel tiles of unequal width
    (17, 16, 14, 15, 32, 5, 5, 1, 2),
    (4, 6, 1, 40, 17, 1, 3, 1, 1),         # one row
    (24, 4, 6, 70, 8, 3, 2, 1, 0),         # segments of a row
    (5, 40, 13, 11, 65, 1, 1, 2, 0),       # strided 1x1
    (3, 50, 13, 11, 33, 1, 1, 1, 0),       # planes as they lie in memory (fp32): 143 elements
    (1, 130, 3, 3, 129, 1, 1, 1, 0),
    (70, 33, 8, 8, 40, 1, 1, 1, 0),
]
TILES = [0, 128128, 96128, 64256, 64128, 32256, 32128]


def _ref(x, dy, R, S, stride, pad):
    u = F.unfold(x.double(), (R, S), padding=pad, stride=stride)
    dw = torch.matmul(dy.double().flatten(2), u.transpose(1, 2).contiguous()).sum(0)
    return dw.reshape(dy.shape[1], x.shape[1], R, S), dy.double().sum((0, 2, 3))


def _close(got, ref, products, what, dtype):
    f = (2e-8 if dtype == "f32" else 6e-8) * products ** 0.5 + 6e-8
    assert float((got.double().cpu() - ref).norm()) <= f * float(ref.norm()), what


def _run(pa, desc, x, dy, shape, code, beta=0.0, prev=None):
    n = pa.purine_conv_workspace_bytes(pa.PURINE_CONV_BWD_WEIGHT_BIAS, desc, x.shape, shape, code)
    ws = torch.full((max(256, n),), 255, dtype=torch.uint8, device="cuda")
    dw = torch.full(shape, float("nan"), device="cuda") if prev is None else prev[0].clone()
    db = torch.full((shape[0],), float("nan"), device="cuda") if prev is None else prev[1].clone()
    pa.purine_conv_bwd_weight_bias(desc, x, dy, dw, db, beta=beta, ws=ws)
    alone = torch.full(shape, float("nan"), device="cuda") if prev is None else prev[0].clone()
    pa.purine_conv_bwd_weight(desc, x, dy, alone, beta=beta, ws=ws)
    assert torch.equal(dw.view(torch.int32), alone.view(torch.int32))
    return dw, db


def _runs(case, dtype, tile):
    """bf16 planes as they lie in memory have no such kernel, and 130 channels of a 256-column tile no room in LDS."""
    flat = case[5:] == (1, 1, 1, 0)
    return not (flat and (dtype == "bf16" or (case[1] > 128 and tile in (64256, 32256))))


ALL = [(c, d, t) for c in CASES for d in ("f32", "bf16") for t in TILES if _runs(c, d, t)]


@pytest.mark.parametrize("case,dtype,tile", ALL, ids=["x".join(map(str, c)) + "-%s-%d" % (d, t) for c, d, t in ALL])
def test_wgrad_staged(case, dtype, tile):
    import paper_1412_6249_amd as pa
    N, C, H, W, K, R, S, s, p = case
    g = torch.Generator().manual_seed(sum(case) * 5 + 3)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    code = pa.PURINE_F32 if dtype == "f32" else pa.PURINE_BF16
    P, Q = (H + 2 * p - R) // s + 1, (W + 2 * p - S) // s + 1
    x0 = torch.randn((N, C, H, W), generator=g).to(td).cuda()
    dy0 = (torch.randn((N, K, P, Q), generator=g) * 1e-3).to(td).cuda()

    def slice_of(t):                       # images further apart than they are large
        each = t[0].numel()
        ns = (each + 31) // 8 * 8
        wide = torch.full((N * ns + 64,), float("nan"), dtype=td, device="cuda")
        v = torch.as_strided(wide, t.shape, (ns,) + t.stride()[1:], 16)
        v.copy_(t)
        return v

    desc = pa.conv_desc(s, p)
    pa.purine_debug_force_tile(-11, tile)
    try:
        assert pa.purine_conv_route(pa.PURINE_CONV_BWD_WEIGHT, desc, x0.shape, (K, C, R, S), code) == pa.PURINE_ROUTE_INSIDE_LDS
        for x, dy in ((x0, dy0), (slice_of(x0), slice_of(dy0))):
            rw, rb = _ref(x.cpu(), dy.cpu(), R, S, s, p)
            dw, db = _run(pa, desc, x, dy, (K, C, R, S), code)
            _close(dw, rw, N * P * Q, "dw", dtype)
            _close(db, rb, 4 * N * P * Q, "db", "bf16")      # a plain fp32 sum
            dw2, db2 = _run(pa, desc, x, dy, (K, C, R, S), code, 1.0, (dw, db))
            _close(dw2, 2 * rw, N * P * Q, "dw, accumulated", dtype)
            _close(db2, 2 * rb, 4 * N * P * Q, "db, accumulated", "bf16")
    finally:
        pa.purine_debug_force_tile(0, 0)


@pytest.mark.parametrize("case,dtype", [(c, d) for c in [(3, 5, 11, 13, 33, 3, 3, 1, 1), (9, 3, 21, 22, 20, 3, 3, 2, 0), (3, 50, 13, 11, 33, 1, 1, 1, 0)]
                                        for d in ("f32", "bf16") if _runs(c, d, 0)])
def test_infinities(case, dtype):
    """An infinity in x reaches exactly the taps that meet it (also next to rows, bands and images that do not exist), one in dy its row."""
    import paper_1412_6249_amd as pa
    N, C, H, W, K, R, S, s, p = case
    g = torch.Generator().manual_seed(11)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    code = pa.PURINE_F32 if dtype == "f32" else pa.PURINE_BF16
    P, Q = (H + 2 * p - R) // s + 1, (W + 2 * p - S) // s + 1
    x, dy = torch.rand((N, C, H, W), generator=g).to(td) + 0.5, torch.rand((N, K, P, Q), generator=g).to(td) + 0.5
    x[0, 1, H - 1, W - 1] = float("inf")
    x[N - 1, 2, 0, 0] = float("-inf")
    x[1, 0, H // 2, 0] = float("inf")
    dy[N - 1, 4, P - 1, Q - 1] = float("inf")
    rw, rb = _ref(x, dy, R, S, s, p)
    # (the reference multiplies padding and what a tap does not meet by nothing: zero times infinity does not occur there)
    ref = torch.zeros_like(rw)
    xp = F.pad(x.double(), (p, p, p, p))
    for r in range(R):
        for q in range(S):
            t = xp[:, :, r:r + (P - 1) * s + 1:s, q:q + (Q - 1) * s + 1:s]
            ref[:, :, r, q] = (dy.double()[:, :, None] * t[:, None]).sum((0, 3, 4))
    pa.purine_debug_force_tile(-11, 0)
    try:
        assert pa.purine_conv_route(pa.PURINE_CONV_BWD_WEIGHT, pa.conv_desc(s, p), x.shape, (K, C, R, S), code) == pa.PURINE_ROUTE_INSIDE_LDS
        dw, db = _run(pa, pa.conv_desc(s, p), x.cuda(), dy.cuda(), (K, C, R, S), code)
    finally:
        pa.purine_debug_force_tile(0, 0)
    dw, db = dw.cpu().double(), db.cpu().double()
    for got, want in ((dw, ref), (db, rb)):
        assert torch.equal(torch.isnan(got), torch.isnan(want))
        inf = torch.isinf(want)
        assert torch.equal(got[inf], want[inf]) and inf.any()
        ok = torch.isfinite(want)
        np.testing.assert_allclose(got[ok], want[ok], rtol=1e-5)


@pytest.mark.parametrize("which", ["x", "dy", "both"])
@pytest.mark.parametrize("case,dtype", [((12, 192, 28, 28, 16, 1, 1, 1, 0, 256 * 784), "f32"), ((2, 3, 40, 41, 40, 7, 7, 2, 3, 1 << 29), "f32"),
                                        ((9, 3, 21, 23, 40, 7, 7, 2, 3, 1 << 26), "f32"), ((3, 50, 13, 11, 33, 1, 1, 1, 0, 1 << 28), "f32"),
                                        ((2, 3, 41, 41, 40, 7, 7, 2, 3, 1 << 30), "bf16"), ((9, 3, 21, 23, 40, 3, 3, 1, 1, 1 << 27), "bf16")],
                         ids=["wide-concat", "first-layer", "eight-and-one-images", "1x1", "bf16", "bf16-eight-and-one-images"])
def test_views_get_the_bits_of_dense_tensors(case, dtype, which):
    """... also slices of tensors whose images lie 0.25 to 2 GiB apart (2^31 bytes and more in all), beside dense ones whose images begin in
    the middle of a dword; out of the scratch of dense tensors (the query knows no strides)."""
    import paper_1412_6249_amd as pa
    N, C, H, W, K, R, S, s, p, ns = case
    g = torch.Generator().manual_seed(N + K)
    td, code = (torch.float32, pa.PURINE_F32) if dtype == "f32" else (torch.bfloat16, pa.PURINE_BF16)
    P, Q = (H + 2 * p - R) // s + 1, (W + 2 * p - S) // s + 1
    x, dy = torch.randn((N, C, H, W), generator=g).to(td), torch.randn((N, K, P, Q), generator=g).to(td)
    desc = pa.conv_desc(s, p)

    def far(t):
        wide = torch.empty((N - 1) * ns + t[0].numel() + 64, dtype=td, device="cuda")
        v = torch.as_strided(wide, t.shape, (ns,) + t.stride()[1:], 0)
        v.copy_(t)
        return v

    dx, ddy = x.cuda(), dy.cuda()
    vx, vdy = far(x) if which != "dy" else dx, far(dy) if which != "x" else ddy
    hook = 0 if dtype == "f32" else -11
    pa.purine_debug_force_tile(hook, 0)
    try:
        assert pa.purine_conv_route(pa.PURINE_CONV_BWD_WEIGHT, desc, x.shape, (K, C, R, S), code) == pa.PURINE_ROUTE_INSIDE_LDS
        dw, db = _run(pa, desc, vx, vdy, (K, C, R, S), code)
        dw0, db0 = _run(pa, desc, dx, ddy, (K, C, R, S), code)
    finally:
        pa.purine_debug_force_tile(0, 0)
    assert torch.equal(dw, dw0) and torch.equal(db, db0)
    rw, rb = _ref(x, dy, R, S, s, p)
    _close(dw, rw, N * P * Q, "dw", dtype)
    _close(db, rb, 4 * N * P * Q, "db", "bf16")
