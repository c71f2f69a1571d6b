"""Second passes that add the splits of a product with many elements: four elements per thread, one where the count is no multiple of
four, the last workgroup not full, counts on both sides of 2^17, accumulation, the bias gradient beside the weight gradient, and the
bf16 fully-connected forward pass, which adds its bias and rounds there. Against float64 sums on the CPU.

Bound: products of bf16 are exact in fp32, so an fp32 chain's rounding (2.7e-8 * sqrt(products); twice that and the last rounding are
allowed) is the whole error, also of the fp32 layers; bf16 results are rounded once (2^-9)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _close(got, ref, products, rounded, what):
    f = 2 ** -8.5 if rounded else 6e-8 * products ** 0.5 + 6e-8
    assert float((got.double().cpu() - ref).norm()) <= f * float(ref.norm()), what


def _ws(n):
    return torch.full((max(256, n),), 255, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("N,C,K", [(37, 1030, 3600), (37, 1031, 3601), (32, 2048, 4096), (31, 2048, 4095), (304, 517, 515), (512, 256, 512), (505, 701, 300)])
def test_fc(N, C, K):
    import paper_1412_6249_amd as pa
    g = torch.Generator().manual_seed(N + C + K)
    rnd = lambda *s: torch.randn(s, generator=g).to(torch.bfloat16)
    x, w, b, dy = rnd(N, C), (rnd(K, C) * C ** -0.5), rnd(K), rnd(N, K)
    d = [t.cuda() for t in (x, w, b, dy)]
    ws = lambda p: _ws(pa.purine_fc_workspace_bytes(p, N, C, K, pa.PURINE_BF16))
    for bias in (d[2], None):
        y = torch.full((N, K), float("nan"), dtype=torch.bfloat16, device="cuda")
        pa.purine_fc_fwd(d[0], d[1], bias, y, ws=ws(pa.PURINE_CONV_FWD))
        _close(y, x.double() @ w.double().t() + (b.double() if bias is not None else 0), C, True, "y")
    dw, db = torch.full((K, C), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
    pa.purine_fc_bwd_weight(d[0], d[3], dw, db, ws=ws(pa.PURINE_CONV_BWD_WEIGHT))
    _close(dw, dy.double().t() @ x.double(), N, False, "dw")
    _close(db, dy.double().sum(0), N, False, "db")
    prev = dw.clone()
    pa.purine_fc_bwd_weight(d[0], d[3], dw, None, beta=1.0, ws=ws(pa.PURINE_CONV_BWD_WEIGHT))
    _close(dw, 2 * dy.double().t() @ x.double(), N, False, "dw + dw")
    assert not torch.equal(dw, prev)


def _both(pa, call):
    """The same call with the kernels of few splits and with the ones that they stand for."""
    out = []
    for hook in (0, -13):
        pa.purine_debug_force_tile(hook, 0)
        try:
            out.append(call())
        finally:
            pa.purine_debug_force_tile(0, 0)
    for a, b in zip(*out):
        assert torch.equal(a.view(torch.int32 if a.dtype == torch.float32 else torch.int16), b.view(torch.int32 if b.dtype == torch.float32 else torch.int16))
    return out[0]


@pytest.mark.parametrize("N,C,K", [(128, 4608, 2048), (300, 4099, 1021), (512, 1024, 512)])
def test_fc_forward_bits(N, C, K):
    """The bias and the rounding in either second pass."""
    import paper_1412_6249_amd as pa
    assert pa.purine_fc_route(pa.PURINE_CONV_FWD, N, C, K, pa.PURINE_BF16) == pa.PURINE_ROUTE_OTHER
    g = torch.Generator().manual_seed(N + C + K)
    x, w, b = (torch.randn(s, generator=g).to(torch.bfloat16).cuda() for s in ((N, C), (K, C), (K,)))
    ws = _ws(pa.purine_fc_workspace_bytes(pa.PURINE_CONV_FWD, N, C, K, pa.PURINE_BF16))

    def call():
        out = []
        for bias in (b, None):
            out.append(torch.full((N, K), float("nan"), dtype=torch.bfloat16, device="cuda"))
            pa.purine_fc_fwd(x, w, bias, out[-1], ws=ws)
        return out
    _close(_both(pa, call)[0], x.double().cpu() @ w.double().cpu().t() + b.double().cpu(), C, True, "y")


@pytest.mark.parametrize("N,C,H,K", [(12, 400, 14, 360), (12, 401, 14, 357), (9, 332, 16, 396), (5, 512, 13, 256)])
def test_weight_gradient_bits(N, C, H, K):
    """... also of gradients that are minus zero and stay it or not."""
    import paper_1412_6249_amd as pa
    g = torch.Generator().manual_seed(N + C + K)
    x, dy = (torch.randn(N, c, H, H, generator=g).to(torch.bfloat16).cuda() for c in (C, K))
    dy[:, ::7] = 0.0
    desc = pa.conv_desc(1, 0)
    assert pa.purine_conv_route(pa.PURINE_CONV_BWD_WEIGHT, desc, x.shape, (K, C, 1, 1), pa.PURINE_BF16) == pa.PURINE_ROUTE_OTHER
    ws = _ws(pa.purine_conv_workspace_bytes(pa.PURINE_CONV_BWD_WEIGHT_BIAS, desc, x.shape, (K, C, 1, 1), pa.PURINE_BF16))
    before = torch.randn((K, C, 1, 1), generator=g).cuda()
    before[:, ::3] = -0.0

    def call():
        dw, db, more = torch.empty_like(before), torch.empty(K, device="cuda"), before.clone()
        pa.purine_conv_bwd_weight_bias(desc, x, dy, dw, db, ws=ws)
        pa.purine_conv_bwd_weight(desc, x, dy, more, beta=1.0, ws=ws)
        return dw, db, more
    _both(pa, call)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,C,H,K", [(12, 400, 14, 360), (12, 401, 14, 357), (9, 331, 17, 396), (9, 332, 16, 396), (5, 512, 13, 256)])
def test_1x1_weight_and_bias(N, C, H, K, dtype):
    import paper_1412_6249_amd as pa
    g = torch.Generator().manual_seed(N + C + K)
    td, code = (torch.float32, pa.PURINE_F32) if dtype == "f32" else (torch.bfloat16, pa.PURINE_BF16)
    x, dy = (torch.randn(N, c, H, H, generator=g).to(td) for c in (C, K))
    rows = lambda t: t.double().permute(1, 0, 2, 3).flatten(1)
    rw, rb = (rows(dy) @ rows(x).t()).reshape(K, C, 1, 1), rows(dy).sum(1)
    desc = pa.conv_desc(1, 0)
    n = pa.purine_conv_workspace_bytes(pa.PURINE_CONV_BWD_WEIGHT_BIAS, desc, x.shape, (K, C, 1, 1), code)
    dw, db = torch.full((K, C, 1, 1), float("nan"), device="cuda"), torch.full((K,), float("nan"), device="cuda")
    pa.purine_conv_bwd_weight_bias(desc, x.cuda(), dy.cuda(), dw, db, ws=_ws(n))
    _close(dw, rw, N * H * H, False, "dw")
    _close(db, rb, N * H * H, False, "db")
    alone = torch.full_like(dw, float("nan"))
    pa.purine_conv_bwd_weight(desc, x.cuda(), dy.cuda(), alone, ws=_ws(n))
    assert torch.equal(alone, dw)
    pa.purine_conv_bwd_weight_bias(desc, x.cuda(), dy.cuda(), dw, db, beta=1.0, ws=_ws(n))
    _close(dw, 2 * rw, N * H * H, False, "dw + dw")
    _close(db, 2 * rb, N * H * H, False, "db + db")
