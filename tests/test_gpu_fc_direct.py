"""Fully-connected passes in one launch: row and column tiles that are not full, reductions of one step, of a step that is not whole and
of the lengths at which the number of wavefronts changes (4 and 32 steps of 16, in each pass and type), rows of odd length (bf16 rows that begin in the middle of a
dword), no bias, accumulation, infinities. Against float64 sums on the CPU.

Bound: fp32 three quarters of an fp32 chain's 2.7e-8 * sqrt(products) and the last rounding; bf16 results are rounded once (2^-9), its fp32
gradients are an fp32 chain's."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# images, inputs, outputs
CASES = [(1, 64, 10), (3, 65, 33), (16, 16, 16), (17, 70, 31), (5, 512, 40), (9, 527, 31), (33, 300, 129), (65, 129, 64), (64, 64, 63), (80, 513, 97),
         (2, 1000, 100), (600, 40, 33), (5, 40, 600)]


@pytest.fixture
def small():
    """... whatever the dispatch would do with a size."""
    import paper_1412_6249_amd as pa
    pa.purine_debug_force_tile(-12, 0)
    yield
    pa.purine_debug_force_tile(0, 0)


def _data(pa, case, dtype):
    N, C, K = case
    g = torch.Generator().manual_seed(N * 7 + C * 3 + K)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    rnd = lambda *s: torch.randn(s, generator=g)
    t = {"x": rnd(N, C).to(td), "w": (rnd(K, C) * C ** -0.5).to(td), "b": rnd(K).to(td), "dy": rnd(N, K).to(td)}
    code = pa.PURINE_F32 if dtype == "f32" else pa.PURINE_BF16
    ws = lambda p: torch.full((max(256, pa.purine_fc_workspace_bytes(p, N, C, K, code)),), 255, dtype=torch.uint8, device="cuda")
    return t, {k: v.cuda() for k, v in t.items()}, ws, td


def _close(got, ref, products, rounded, what):
    f = 2 ** -8.5 if rounded else 2e-8 * products ** 0.5 + 6e-8
    assert float((got.double().cpu() - ref).norm()) <= f * float(ref.norm()), what


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_fc_direct(case, dtype, small):
    import paper_1412_6249_amd as pa
    N, C, K = case
    t, d, ws, td = _data(pa, case, dtype)
    assert [pa.purine_fc_route(p, N, C, K, pa.PURINE_F32 if dtype == "f32" else pa.PURINE_BF16) for p in range(3)] == [pa.PURINE_ROUTE_SMALL_LAUNCH] * 3
    r = {k: v.double() for k, v in t.items()}
    nan = lambda *s, dt=td: torch.full(s, float("nan"), dtype=dt, device="cuda")
    for b in (d["b"], None):
        y = nan(N, K)
        pa.purine_fc_fwd(d["x"], d["w"], b, y, ws=ws(pa.PURINE_CONV_FWD))
        _close(y, r["x"] @ r["w"].t() + (r["b"] if b is not None else 0), C, dtype == "bf16", "y")
    dx = nan(N, C)
    pa.purine_fc_bwd_data(d["dy"], d["w"], dx, ws=ws(pa.PURINE_CONV_BWD_DATA))
    _close(dx, r["dy"] @ r["w"], K, dtype == "bf16", "dx")
    rw, rb = r["dy"].t() @ r["x"], r["dy"].sum(0)
    dw, db = nan(K, C, dt=torch.float32), nan(K, dt=torch.float32)
    pa.purine_fc_bwd_weight(d["x"], d["dy"], dw, db, ws=ws(pa.PURINE_CONV_BWD_WEIGHT))
    _close(dw, rw, N, False, "dw")
    assert float((db.double().cpu() - rb).norm()) <= 1e-7 * float(r["dy"].norm()) * N ** 0.5
    alone = nan(K, C, dt=torch.float32)
    pa.purine_fc_bwd_weight(d["x"], d["dy"], alone, None, ws=ws(pa.PURINE_CONV_BWD_WEIGHT))
    assert torch.equal(alone, dw)
    db0 = db.clone()
    pa.purine_fc_bwd_weight(d["x"], d["dy"], dw, db, beta=1.0, ws=ws(pa.PURINE_CONV_BWD_WEIGHT))
    assert torch.equal(dw, alone + alone) and torch.equal(db, db0 + db0)


@pytest.mark.parametrize("over", ["x", "w"])
@pytest.mark.parametrize("N,C,K", [(9, 64, 64), (64, 40, 64), (33, 35, 35)])
def test_bf16_forward_over_its_operands(N, C, K, over):
    """y in the place of x or w: the product is complete before it is written."""
    import paper_1412_6249_amd as pa
    t, d, ws, td = _data(pa, (N, C, K), "bf16")
    y = torch.as_strided(torch.cat([d[over].flatten(), torch.zeros(N * K, dtype=td, device="cuda")]), (N, K), (K, 1), 0)
    d[over] = torch.as_strided(y, d[over].shape, (C, 1), 0)
    pa.purine_fc_fwd(d["x"], d["w"], d["b"], y, ws=ws(pa.PURINE_CONV_FWD))
    _close(y, t["x"].double() @ t["w"].double().t() + t["b"].double(), C, True, "y")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,K", [(256, 17), (257, 16), (511, 1), (512, 40), (513, 65), (961, 15), (5000, 33)])
def test_bias_gradient_of_many_images(N, K, dtype):
    """On both sides of the row count from which a workgroup takes 16 columns, rows that do not fill its last round; never read past the end."""
    import paper_1412_6249_amd as pa
    t, d, ws, td = _data(pa, (N, 24, K), dtype)
    rb = t["dy"].double().sum(0)
    dw, db = torch.empty(K, 24, device="cuda"), torch.full((K,), float("nan"), device="cuda")
    pa.purine_debug_force_tile(-13, 0)
    try:
        pa.purine_fc_bwd_weight(d["x"], d["dy"], dw, db, ws=ws(pa.PURINE_CONV_BWD_WEIGHT))
        first = db.clone()
        pa.purine_fc_bwd_weight(d["x"], d["dy"], dw, db, beta=1.0, ws=ws(pa.PURINE_CONV_BWD_WEIGHT))
    finally:
        pa.purine_debug_force_tile(0, 0)
    assert float((first.double().cpu() - rb).norm()) <= 1e-7 * float(t["dy"].double().norm()) * N ** 0.5
    assert torch.equal(db, first + first)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_infinities(dtype, small):
    """At the ends of rows, where the next row's elements are loaded along with them."""
    import paper_1412_6249_amd as pa
    N, C, K = 9, 67, 35
    t, d, ws, td = _data(pa, (N, C, K), dtype)
    t = {k: v.abs() + 0.5 for k, v in t.items()}
    t["x"][1, 0] = float("inf")
    t["x"][4, C - 1] = float("-inf")
    t["w"][3, 0] = float("inf")
    t["dy"][5, 0] = float("inf")
    t["dy"][6, K - 1] = float("-inf")
    d = {k: v.cuda() for k, v in t.items()}
    r = {k: v.double() for k, v in t.items()}
    y, dx = torch.empty(N, K, dtype=td, device="cuda"), torch.empty(N, C, dtype=td, device="cuda")
    dw, db = torch.empty(K, C, device="cuda"), torch.empty(K, device="cuda")
    pa.purine_fc_fwd(d["x"], d["w"], d["b"], y, ws=ws(pa.PURINE_CONV_FWD))
    pa.purine_fc_bwd_data(d["dy"], d["w"], dx, ws=ws(pa.PURINE_CONV_BWD_DATA))
    pa.purine_fc_bwd_weight(d["x"], d["dy"], dw, db, ws=ws(pa.PURINE_CONV_BWD_WEIGHT))
    for got, want in ((y, r["x"] @ r["w"].t() + r["b"]), (dx, r["dy"] @ r["w"]), (dw, r["dy"].t() @ r["x"]), (db, r["dy"].sum(0))):
        got = got.double().cpu()
        assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(got[torch.isinf(want)], want[torch.isinf(want)])
        ok = torch.isfinite(want)
        assert ok.any() and torch.allclose(got[ok], want[ok], rtol=2 ** -8 if got is not dw else 1e-5)
