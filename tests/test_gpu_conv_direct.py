"""Forward and backward-data of small launches in one kernel: row and pixel tiles that are not full, reductions of one step and of the lengths
at which the number of wavefronts changes, ends of the reduction inside a step, bf16 filter rows that begin in the middle of a
dword, strides (also beyond the filter), padding, filters of unequal sides, channel-slice views, bias, ReLU, mask, accumulation, infinities.
Against float64 sums on the CPU.

Bound: fp32 three quarters of an fp32 chain's 2.7e-8 * sqrt(products) and the last roundings; bf16 results are rounded once."""
import pytest
import torch
import torch.nn.functional as F

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad
CASES = [
    (1, 1, 3, 3, 1, 3, 3, 1, 1),
    (2, 3, 8, 8, 8, 3, 3, 1, 1),
    (1, 16, 7, 5, 33, 1, 1, 1, 0),
    (3, 7, 9, 11, 20, 3, 3, 2, 1),
    (2, 5, 10, 10, 40, 5, 5, 2, 2),
    (1, 4, 12, 13, 6, 2, 3, 3, 0),         # stride beyond the filter in one direction
    (2, 3, 30, 31, 35, 11, 11, 4, 5),
    (2, 38, 8, 9, 42, 3, 3, 1, 1),
    (5, 29, 6, 6, 64, 3, 3, 1, 0),         # 261 products: the last step holds five
    (1, 57, 5, 4, 31, 5, 5, 1, 2),
    (4, 17, 6, 7, 18, 1, 1, 2, 0),
    (1, 100, 4, 4, 70, 3, 3, 1, 1),
    (1, 512, 7, 7, 24, 3, 3, 1, 1),        # 4608 products forward, and
    (1, 24, 7, 7, 910, 3, 3, 1, 1),        # 8190 backward: tables of more than 64 KB
]


def _slice_of(t):                          # images further apart than they are large
    each = t[0].numel()
    ns = (each + 31) // 8 * 8
    wide = torch.full((t.shape[0] * ns + 64,), float("nan"), dtype=t.dtype, device="cuda")
    v = torch.as_strided(wide, t.shape, (ns,) + t.stride()[1:], 16)
    v.copy_(t)
    return v


def _close(got, ref, products, dtype, what):
    f = 2 ** -8.5 if dtype == "bf16" else 2e-8 * products ** 0.5 + 1e-7
    assert float((got.double().cpu() - ref).norm()) <= f * float(ref.norm()), what


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_conv_direct(case, dtype):
    import paper_1412_6249_amd as pa
    N, C, H, W, K, R, S, s, p = case
    g = torch.Generator().manual_seed(sum(case) * 3 + 1)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    code = pa.PURINE_F32 if dtype == "f32" else pa.PURINE_BF16
    x, w, b = (torch.randn(sh, generator=g).to(td) for sh in ((N, C, H, W), (K, C, R, S), (K,)))
    xd = x.double().requires_grad_()
    y = F.conv2d(xd, w.double(), b.double(), stride=s, padding=p)
    dy = torch.randn(y.shape, generator=g).to(td)
    dx, = torch.autograd.grad(y, xd, dy.double())
    y = y.detach()
    desc = pa.conv_desc(s, p)
    ws = lambda which: torch.empty(max(256, pa.purine_conv_workspace_bytes(which, desc, x.shape, w.shape, code)), dtype=torch.uint8, device="cuda")
    tw, tb = w.cuda(), b.cuda()
    pa.purine_debug_force_tile(-12, 0)
    try:
        assert [pa.purine_conv_route(q, desc, x.shape, w.shape, code) for q in (0, 1)] == [pa.PURINE_ROUTE_SMALL_LAUNCH] * 2
        for view in (lambda t: t.cuda(), _slice_of):
            tx, tdy = view(x.cuda()), view(dy.cuda())
            out, odx = view(torch.full(y.shape, float("nan"), dtype=td, device="cuda")), view(torch.full(x.shape, float("nan"), dtype=td, device="cuda"))
            pa.purine_conv_fwd_bias_relu(desc, tx, tw, tb, out, relu=True, ws=ws(pa.PURINE_CONV_FWD))
            _close(out, F.relu(y), C * R * S, dtype, "forward with bias and ReLU")
            pa.purine_conv_fwd(desc, tx, tw, out, ws=ws(pa.PURINE_CONV_FWD))
            _close(out, y - b.double().view(1, -1, 1, 1), C * R * S, dtype, "forward")
            pa.purine_conv_bwd_data(desc, tdy, tw, odx, ws=ws(pa.PURINE_CONV_BWD_DATA))
            _close(odx, dx, K * R * S, dtype, "backward-data")
            pa.purine_conv_bwd_data(desc, tdy, tw, odx, beta=1.0, ws=ws(pa.PURINE_CONV_BWD_DATA))
            _close(odx, 2 * dx, K * R * S, dtype, "accumulated")
            pa.purine_conv_bwd_data_relu(desc, tdy, tw, tx, odx, ws=ws(pa.PURINE_CONV_BWD_DATA))
            _close(odx, dx * (x.double() > 0), K * R * S, dtype, "through the mask")
    finally:
        pa.purine_debug_force_tile(0, 0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(2, 3, 8, 8, 8, 3, 3, 1, 1), (2, 5, 10, 10, 40, 5, 5, 2, 2), (2, 38, 8, 9, 42, 3, 3, 1, 1)], ids=["2", "8", "16"])
def test_far_images(case, dtype):
    """Images 2^31 bytes apart, for each number of wavefronts: the bits of dense tensors."""
    import paper_1412_6249_amd as pa
    N, C, H, W, K, R, S, s, p = case
    g = torch.Generator().manual_seed(sum(case))
    td, code, ns = (torch.float32, pa.PURINE_F32, 1 << 29) if dtype == "f32" else (torch.bfloat16, pa.PURINE_BF16, 1 << 30)
    desc = pa.conv_desc(s, p)
    x, w = (torch.randn(sh, generator=g).to(td).cuda() for sh in ((N, C, H, W), (K, C, R, S)))
    dy = torch.randn(pa.purine_conv_out_shape(desc, x.shape, w.shape), generator=g).to(td).cuda()
    ws = lambda which: torch.empty(max(256, pa.purine_conv_workspace_bytes(which, desc, x.shape, w.shape, code)), dtype=torch.uint8, device="cuda")

    def far(t):
        v = torch.as_strided(torch.empty((N - 1) * ns + t[0].numel() + 64, dtype=td, device="cuda"), t.shape, (ns,) + t.stride()[1:], 0)
        v.copy_(t)
        return v

    pa.purine_debug_force_tile(-12, 0)
    try:
        y, dx = torch.empty_like(dy), torch.empty_like(x)
        pa.purine_conv_fwd(desc, x, w, y, ws=ws(pa.PURINE_CONV_FWD))
        pa.purine_conv_bwd_data(desc, dy, w, dx, ws=ws(pa.PURINE_CONV_BWD_DATA))
        y2, dx2 = far(torch.zeros_like(dy)), far(torch.zeros_like(x))
        pa.purine_conv_fwd(desc, far(x), w, y2, ws=ws(pa.PURINE_CONV_FWD))
        pa.purine_conv_bwd_data(desc, far(dy), w, dx2, ws=ws(pa.PURINE_CONV_BWD_DATA))
    finally:
        pa.purine_debug_force_tile(0, 0)
    assert torch.equal(y2, y) and torch.equal(dx2, dx)
    _close(y, F.conv2d(x.cpu().double(), w.cpu().double(), stride=s, padding=p), C * R * S, dtype, "forward")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("stride", [1, 2])
def test_infinities(stride, dtype):
    """Infinite activations and gradients reach exactly the outputs whose taps meet them (a strided backward pass meets none of the others)."""
    import paper_1412_6249_amd as pa
    N, C, H, W, K, R = 2, 5, 9, 9, 6, 3
    g = torch.Generator().manual_seed(4)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    code = pa.PURINE_F32 if dtype == "f32" else pa.PURINE_BF16
    x, w = torch.rand((N, C, H, W), generator=g).to(td) + 0.5, torch.rand((K, C, R, R), generator=g).to(td) + 0.5
    x[0, 1, 4, 4] = float("inf")
    x[1, 2, 0, 0] = float("-inf")
    finite = torch.where(torch.isinf(x), torch.zeros_like(x), x)
    P = (H - R) // stride + 1
    dy = torch.rand((N, K, P, P), generator=g).to(td) + 0.5
    dy[1, 3, 1, 2] = float("inf")
    dyf = torch.where(torch.isinf(dy), torch.zeros_like(dy), dy)
    met = lambda t: F.conv2d(torch.isinf(t).double().sum(1, keepdim=True), torch.ones(1, 1, R, R, dtype=torch.double), stride=stride) > 0
    y = F.conv2d(finite.double(), w.double(), stride=stride)
    hit = met(x).expand(-1, K, -1, -1)
    back = lambda t: F.conv_transpose2d(t, w.double(), stride=stride, output_padding=(H - R) % stride)
    dx = back(dyf.double())
    hit_dx = F.conv_transpose2d(torch.isinf(dy).double().sum(1, keepdim=True), torch.ones(1, 1, R, R, dtype=torch.double), stride=stride,
                                output_padding=(H - R) % stride).expand(-1, C, -1, -1) > 0
    desc = pa.conv_desc(stride, 0)
    ws = lambda which: torch.empty(max(256, pa.purine_conv_workspace_bytes(which, desc, x.shape, w.shape, code)), dtype=torch.uint8, device="cuda")
    out, odx = torch.empty(y.shape, dtype=td, device="cuda"), torch.empty(x.shape, dtype=td, device="cuda")
    pa.purine_debug_force_tile(-12, 0)
    try:
        pa.purine_conv_fwd(desc, x.cuda(), w.cuda(), out, ws=ws(pa.PURINE_CONV_FWD))
        pa.purine_conv_bwd_data(desc, dy.cuda(), w.cuda(), odx, ws=ws(pa.PURINE_CONV_BWD_DATA))
    finally:
        pa.purine_debug_force_tile(0, 0)
    for got, ref, h in ((out, y, hit), (odx, dx, hit_dx)):
        got = got.double().cpu()
        assert torch.equal(torch.isinf(got), h) and not torch.isnan(got).any()
        assert torch.allclose(got[~h], ref[~h], rtol=2 ** -8 if dtype == "bf16" else 1e-5)
