"""fp32 1x1 layers on bf16 parts split in registers: strips and row tiles that are not full, channel counts that are
not whole groups or packets, one pixel, few and many strips per wavefront, strided forward gathers, channel-slice
views, an accumulating and a masked backward pass, infinities and NaN. Against float64 sums on the CPU.

Bound: the three products left out are below 2^-24 of |a||b| each. An fp32 chain of n products rounds by 2.7e-8 * sqrt(n), this kernel's
sums by a third to a half of that; three quarters of it, and two roundings at the end, are allowed: a lost part, or a product of the six,
is several times as much in sums of any length."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

pytestmark = pytest.mark.gpu

# N, C, H, W, K, stride
CASES = [
    (1, 16, 1, 1, 40, 1),
    (2, 17, 5, 7, 33, 1),
    (3, 96, 13, 13, 96, 1),
    (1, 45, 9, 31, 65, 1),
    (5, 231, 6, 10, 49, 1),        # rows of W that are no whole packets
    (2, 500, 8, 8, 40, 1),         # 32 steps; 64-row tiles do not fit LDS
    (40, 20, 57, 59, 24, 1),       # several strips per wavefront
    (2, 36, 11, 9, 70, 2),
    (1, 24, 10, 13, 20, 3),
    (4, 30, 6, 6, 10, 1),          # ten gathered channels backward
]


def _close(got, ref, products, what):
    got, ref = got.double().cpu(), ref.double()
    assert float((got - ref).norm()) <= (2e-8 * products ** 0.5 + 6e-8) * float(ref.norm()), what


@pytest.mark.parametrize("tm", [0, 1, 2])
@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_1x1_split(case, tm):
    import paper_1412_6249_amd as pa
    N, C, H, W, K, s = case
    g = torch.Generator().manual_seed(sum(case) * 7 + 1)
    rnd = lambda *shape: torch.randn(shape, generator=g)
    x, w, b = rnd(N, C, H, W).clamp(min=0), rnd(K, C, 1, 1) * 0.2, rnd(K)
    y = F.conv2d(x.double(), w.double(), b.double(), stride=s)
    dy = rnd(*y.shape)
    dx = F.conv_transpose2d(dy.double(), w.double(), stride=s,
                            output_padding=((H - 1) % s, (W - 1) % s))
    d = lambda t: t.cuda().contiguous()
    tx, tw, tb, tdy = d(x), d(w), d(b), d(dy)
    desc = pa.conv_desc(s, 0)
    pa.purine_debug_force_tile(-10, tm)
    try:
        ws = lambda p: torch.empty(max(256, pa.purine_conv_workspace_bytes(p, desc, tx.shape, tw.shape, 0)), dtype=torch.uint8, device="cuda")
        out = torch.full(tuple(y.shape), float("nan"), device="cuda")
        pa.purine_conv_fwd_bias_relu(desc, tx, tw, tb, out, relu=True, ws=ws(pa.PURINE_CONV_FWD))
        _close(out, F.relu(y), C, "forward with bias and ReLU")
        pa.purine_conv_fwd(desc, tx, tw, out, ws=ws(pa.PURINE_CONV_FWD))
        _close(out, y - b.double().view(1, -1, 1, 1), C, "forward")
        wsb = ws(pa.PURINE_CONV_BWD_DATA)
        tdx = torch.full(tuple(x.shape), float("nan"), device="cuda")
        pa.purine_conv_bwd_data(desc, tdy, tw, tdx, ws=wsb)
        _close(tdx, dx, K, "backward-data")
        pa.purine_conv_bwd_data(desc, tdy, tw, tdx, beta=1.0, ws=wsb)
        _close(tdx, 2 * dx, K, "backward-data, accumulating")
        pa.purine_conv_bwd_data_relu(desc, tdy, tw, tx, tdx, ws=wsb)
        _close(tdx, dx * (x > 0), K, "backward-data through the mask")
    finally:
        pa.purine_debug_force_tile(0, 0)


def test_1x1_split_views():
    """Output and input channel slices of wider tensors; what lies around them stays."""
    import paper_1412_6249_amd as pa
    N, C, H, W, K = 3, 24, 7, 12, 40
    g = torch.Generator().manual_seed(3)
    big = torch.randn((N, C + 16, H, W), generator=g).cuda()
    w = (torch.randn((K, C, 1, 1), generator=g) * 0.2).cuda()
    cat = torch.full((N, K + 24, H, W), 5.0, device="cuda")
    desc = pa.conv_desc(1, 0)
    ref = F.conv2d(big[:, 8:8 + C].cpu().double(), w.cpu().double())
    for tm in (1, 2):
        pa.purine_debug_force_tile(-10, tm)
        try:
            pa.purine_conv_fwd(desc, big[:, 8:8 + C], w, cat[:, 16:16 + K], ws=torch.empty(1 << 20, dtype=torch.uint8, device="cuda"))
        finally:
            pa.purine_debug_force_tile(0, 0)
        _close(cat[:, 16:16 + K], ref, C, "view")
        assert bool((cat[:, :16] == 5).all()) and bool((cat[:, 16 + K:] == 5).all())


@pytest.mark.parametrize("tm", [1, 2])
def test_1x1_split_special_values(tm):
    """Infinities, NaN and numbers too large for the split come out as in a plain fp32 sum, everything else undisturbed."""
    import paper_1412_6249_amd as pa
    N, C, H, W, K = 2, 40, 6, 9, 70
    g = torch.Generator().manual_seed(11)
    x, w = torch.randn((N, C, H, W), generator=g), torch.randn((K, C, 1, 1), generator=g)
    x[0, 3, 2, 5], x[1, 39, 0, 0], x[1, 7, 5, 8], x[0, 1, 1, 1] = float("inf"), float("nan"), -3e38, 2.0 ** 113
    w[69, 0, 0, 0], w[5, 20, 0, 0] = float("-inf"), 2.0 ** 100
    ref = F.conv2d(x.double(), w.double()).float()                 # out of range where the fp32 result is
    out = torch.empty((N, K, H, W), device="cuda")
    pa.purine_debug_force_tile(-10, tm)
    try:
        pa.purine_conv_fwd(pa.conv_desc(1, 0), x.cuda(), w.cuda(), out, ws=torch.empty(1 << 20, dtype=torch.uint8, device="cuda"))
    finally:
        pa.purine_debug_force_tile(0, 0)
    out = out.cpu()
    assert torch.equal(out.isnan(), ref.isnan())
    fin = ref.isfinite() & (ref.abs() < 1e38)
    assert torch.equal(out.isinf() & ref.isinf(), ref.isinf())
    err = (out - ref)[fin].double().abs() / (F.conv2d(x.double().abs().nan_to_num(0, 0, 0), w.double().abs().nan_to_num(0, 0, 0)))[fin]
    assert float(err.max()) <= 40 * 2.0 ** -24                     # one rounding per addition
