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
