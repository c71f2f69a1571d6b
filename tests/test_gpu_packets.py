"""The fp32 convolutions that run on bf16 parts (three per operand, six products): at the edges of their tiles, reduction steps and splits, in every form the operators have, against the oracle and
against the general fp32 kernels (reached by switching raw buffer loads off, which the packed kernels
need). The split must not cost precision: its error against fp64 may not exceed the general kernels'."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad. What is at an edge: one row past a 16- / 32- / 96- / 128-row tile,
# channel counts on either side of a 16-channel step, pixel counts on either side of a tile, tiles that
# cross several images, rows so wide that the LDS patch is cut into bands (a ragged last one), a long
# reduction over few pixels (split over workgroups), unequal filter and image sides, strides
# (phase-folded backward-data) and filters that fit inside one stride step
CASES = [(2, 16, 9, 9, 17, 3, 3, 1, 1), (2, 233, 9, 11, 45, 3, 3, 1, 1), (3, 17, 16, 8, 129, 2, 3, 1, (1, 0)),
         (1, 256, 6, 6, 40, 3, 3, 1, 1), (1, 130, 5, 23, 64, 1, 5, 1, (0, 2)), (4, 31, 27, 29, 96, 3, 3, 2, 1),
         (2, 24, 14, 11, 33, 5, 4, (3, 2), (2, 1)), (5, 96, 13, 13, 97, 3, 3, 1, 1), (8, 64, 28, 28, 33, 3, 3, 1, 1),
         (60, 17, 4, 3, 20, 3, 3, 1, 1), (1, 24, 33, 141, 40, 3, 3, 1, 1), (1, 16, 9, 300, 18, 1, 2, 1, 0),
         (3, 40, 29, 31, 70, 5, 5, 1, 2), (2, 48, 15, 15, 32, 2, 2, 2, 0), (1, 16, 70, 70, 24, 7, 7, 1, 3)]


def _general(pa, on):
    pa.purine_debug_force_tile(0, -1 if on else 0)


def _forced(pa, route):
    """route: "auto", "patch" (split in LDS), "packets" (packed parts), "patch_f32" (forward: the LDS kernel
    with fp32 products) or "general" (fp32 MFMA kernels)."""
    pa.purine_debug_force_tile(*{"auto": (0, 0), "patch": (-6, 0), "packets": (-7, 0), "patch_f32": (-8, 0), "general": (0, -1)}[route])


def _run(pa, case, x, w, b, dy, act, prev):
    """y (bias + ReLU), y (plain), dx, dx accumulated onto prev, dx through the mask; and the scratch sizes."""
    import torch
    from gpu_util import to_dev, workspace, to_host, DEV
    desc = pa.conv_desc(case[7], case[8])
    need = [pa.purine_conv_workspace_bytes(k, desc, x.shape, w.shape, pa.PURINE_F32) for k in (0, 1)]
    wf, wd = (workspace(n) for n in need)
    tx, tw, tb, tdy, tact = (to_dev(a) for a in (x, w, b, dy, act))
    y, yp = (torch.full(dy.shape, float("nan"), device=DEV) for _ in range(2))
    dx, dm = (torch.full(x.shape, float("nan"), device=DEV) for _ in range(2))
    da = to_dev(prev)
    pa.purine_conv_fwd_bias_relu(desc, tx, tw, tb, y, relu=True, ws=wf)
    pa.purine_conv_fwd(desc, tx, tw, yp, ws=wf)
    pa.purine_conv_bwd_data(desc, tdy, tw, dx, ws=wd)
    pa.purine_conv_bwd_data(desc, tdy, tw, da, beta=1.0, ws=wd)
    pa.purine_conv_bwd_data_relu(desc, tdy, tw, tact, dm, ws=wd)
    torch.cuda.synchronize()
    return [to_host(t) for t in (y, yp, dx, da, dm)], need


def _inputs(case, seed=5):
    N, C, H, W, K, R, S, stride, pad = case
    rs = np.random.default_rng(seed)
    f = lambda *s: rs.standard_normal(s).astype(np.float32)
    P, Q = oracle.out_shape((N, C, H, W), (K, C, R, S), stride, pad)[2:]
    return f(N, C, H, W), f(K, C, R, S), f(K), f(N, K, P, Q), f(N, C, H, W), f(N, C, H, W)


@pytest.mark.parametrize("case", CASES, ids=str)
def test_split_products_against_the_oracle_and_the_general_kernels(case):
    """All three routes over the same layers. The general kernels' result is what the split ones may not be
    further off the exact one than."""
    import paper_1412_6249_amd as pa
    from gpu_util import rel_l2
    x, w, b, dy, act, prev = _inputs(case)
    stride, pad = case[7], case[8]
    got = {}
    try:
        for route in ("general", "patch", "packets", "patch_f32", "auto"):
            _forced(pa, route)
            got[route], _ = _run(pa, case, x, w, b, dy, act, prev)
    finally:
        _forced(pa, "auto")
    y = oracle.conv_fwd(x, w, stride, pad)
    dx = oracle.conv_bwd_data(dy, w, x.shape, stride, pad)
    refs = (np.maximum(oracle.bias_fwd(y, b), 0), y, dx, dx + prev, np.where(act > 0, dx, 0.0))
    unit = stride == 1
    sh, sw = (stride, stride) if isinstance(stride, int) else stride
    taps_b = -(-case[5] // sh) * -(-case[6] // sw)           # taps of the phase-folded backward pass; one: not for these kernels
    # the fp32 patch kernel adds in the order of the tap kernel's 32x32x2 tiles: the same bits (16-row tiles,
    # which GEMMs of 33 .. 48 and 81 .. 96 rows take, add in another one)
    K = case[4]
    if unit and not (K <= 16 or 33 <= K <= 48 or 81 <= K <= 96):
        assert all(np.array_equal(g, o) for g, o in zip(got["patch_f32"][:2], got["general"][:2])), case
    for route in ("patch", "packets", "patch_f32", "auto"):
        differs = [not np.array_equal(g, o) for g, o in zip(got[route], got["general"])]
        if route == "patch":             # a strided forward gather is not for this one
            assert (differs[1] or not unit) and (differs[2] or taps_b == 1), case
        elif route == "packets":
            assert differs[1] and (differs[2] or taps_b == 1), case
        for name, g, o, r in zip(("y fused", "y", "dx", "dx accumulated", "dx masked"), got[route], got["general"], refs):
            # both round the result once (0.3 * 2^-24 on average); beyond that the split's sums may be no
            # further off than the fp32 MFMA's
            assert rel_l2(g, r) <= max(rel_l2(o, r), 1.0e-7), (route, name, rel_l2(g, r), rel_l2(o, r))
            assert rel_l2(g, r) <= 1e-5, (route, name)


# Channel slices of wider buffers: images further apart than C*H*W. Tiles that cross images, rows cut into bands, a
# strided forward gather with a phase-folded gradient, 33..48 rows
VIEW_CASES = [(7, 32, 10, 9, 40, 3, 3, 1, 1), (1, 24, 12, 150, 64, 3, 3, 1, 1), (3, 52, 15, 16, 132, 5, 5, 1, 2), (4, 36, 17, 16, 24, 3, 3, 2, 1)]


@pytest.mark.parametrize("route", ["patch", "patch_f32", "packets"])
@pytest.mark.parametrize("case", VIEW_CASES, ids=str)
def test_channel_slice_views_give_the_bits_of_dense_tensors(case, route):
    """Inputs, outputs and the ReLU mask as views with a stride of their own: the same bits as dense tensors on the same
    route, and nothing outside the slices written. The gradients of the weights through the packed kernel too."""
    import torch
    import paper_1412_6249_amd as pa
    from gpu_util import to_dev, workspace, to_host, DEV
    N, C, H, W, K, R, S, stride, pad = case
    x, w, b, dy, act, prev = _inputs(case)
    desc = pa.conv_desc(stride, pad)

    def view(a, before=4, after=8):
        """(slice holding a, the buffer around it, which channels are not the slice's); extents keep 16-byte alignment."""
        n, c, h, wd = a.shape
        after += -(before + c + after) % 4
        buf = torch.full((n, before + c + after, h, wd), 7.5, device=DEV)
        v = buf[:, before:before + c]
        v.copy_(to_dev(a))
        return v, buf, [i for i in range(before + c + after) if not before <= i < before + c]

    tw, tb = to_dev(w), to_dev(b)
    nan = lambda s: np.full(s, np.nan, np.float32)
    try:
        _forced(pa, route)
        want, _ = _run(pa, case, x, w, b, dy, act, prev)
        want_w, want_b, _ = _wgrad(pa, case, x, dy, w, b, 0.0)
        ws = [workspace(pa.purine_conv_workspace_bytes(p, desc, x.shape, w.shape, pa.PURINE_F32)) for p in range(4)]
        tx, tdy, tact = view(x), view(dy, 8, 4), view(act, 0, 12)
        out = [view(nan(dy.shape)), view(nan(dy.shape), 0, 4), view(nan(x.shape), 12, 0), view(prev, 4, 4), view(nan(x.shape), 0, 12)]
        dw, db = to_dev(w), to_dev(b)
        pa.purine_conv_fwd_bias_relu(desc, tx[0], tw, tb, out[0][0], relu=True, ws=ws[0])
        pa.purine_conv_fwd(desc, tx[0], tw, out[1][0], ws=ws[0])
        pa.purine_conv_bwd_data(desc, tdy[0], tw, out[2][0], ws=ws[1])
        pa.purine_conv_bwd_data(desc, tdy[0], tw, out[3][0], beta=1.0, ws=ws[1])
        pa.purine_conv_bwd_data_relu(desc, tdy[0], tw, tact[0], out[4][0], ws=ws[1])
        pa.purine_conv_bwd_weight_bias(desc, tx[0], tdy[0], dw, db, ws=ws[3])
        torch.cuda.synchronize()
    finally:
        _forced(pa, "auto")
    for (v, buf, rest), ref in zip(out, want):
        assert np.array_equal(to_host(v.contiguous()), ref)
        assert bool((buf[:, rest] == 7.5).all())
    assert np.array_equal(to_host(dw), want_w) and np.array_equal(to_host(db), want_b)


@pytest.mark.parametrize("route", ["auto", "patch", "patch_f32", "packets"])
def test_grouped_convolution_is_its_groups_on_every_route(route):
    """Two groups as one call (channel slices of x, y, dx) against each group alone on dense tensors: the same bits."""
    import torch
    import paper_1412_6249_amd as pa
    from gpu_util import to_dev, workspace, DEV
    N, C, H, K, R = 24, 96, 27, 96, 5
    g = torch.Generator().manual_seed(9)
    x, w, b, dy = (torch.randn(s, generator=g).to(DEV) for s in ((N, C, H, H), (K, C // 2, R, R), (K,), (N, K, H, H)))
    desc = pa.conv_desc(1, 2)
    full = lambda t: torch.full_like(t, float("nan"))
    y, dx, dw, db, ya, dxa, dwa, dba = (full(t) for t in (dy, x, w, b, dy, x, w, b))
    try:
        _forced(pa, route)
        ws = [workspace(pa.purine_grouped_conv_workspace_bytes(p, desc, 2, x.shape, w.shape, pa.PURINE_F32)) for p in (0, 1, 3)]
        pa.purine_grouped_conv_fwd(desc, 2, x, w, b, y, relu=True, ws=ws[0])
        pa.purine_grouped_conv_bwd_data(desc, 2, dy, w, dx, ws=ws[1])
        pa.purine_grouped_conv_bwd_weight(desc, 2, x, dy, dw, db, ws=ws[2])
        for i in range(2):
            cs, ks = slice(i * C // 2, (i + 1) * C // 2), slice(i * K // 2, (i + 1) * K // 2)
            xi, wi, bi, di = (t.contiguous() for t in (x[:, cs], w[ks], b[ks], dy[:, ks]))
            yi, dxi, dwi, dbi = full(di), full(xi), full(wi), full(bi)
            wsi = [workspace(pa.purine_conv_workspace_bytes(p, desc, xi.shape, wi.shape, pa.PURINE_F32)) for p in (0, 1, 3)]
            pa.purine_conv_fwd_bias_relu(desc, xi, wi, bi, yi, relu=True, ws=wsi[0])
            pa.purine_conv_bwd_data(desc, di, wi, dxi, ws=wsi[1])
            pa.purine_conv_bwd_weight_bias(desc, xi, di, dwi, dbi, ws=wsi[2])
            ya[:, ks], dxa[:, cs], dwa[ks], dba[ks] = yi, dxi, dwi, dbi
        torch.cuda.synchronize()
    finally:
        _forced(pa, "auto")
    assert torch.equal(y, ya) and torch.equal(dx, dxa) and torch.equal(dw, dwa) and torch.equal(db, dba)


# N, C, H, K, R and whether the forward pass keeps the fp32 order of additions: more than 2048 products and 32 or more tiles of
# 128 channels x 256 positions; GEMMs of 33..48 and 81..96 rows then stay on the 16-row tiles of the tap kernel
@pytest.mark.parametrize("case, keeps", [((20, 256, 13, 384, 3), True), ((50, 256, 13, 40, 3), True), ((50, 230, 13, 96, 3), True), ((50, 228, 13, 130, 3), True),
                                         ((50, 227, 13, 130, 3), False), ((20, 83, 13, 384, 5), True), ((20, 81, 13, 384, 5), False),
                                         ((16, 256, 13, 128, 3), False), ((2, 256, 13, 384, 3), False)], ids=str)
def test_which_forward_passes_keep_the_fp32_order(case, keeps):
    """The automatic route of long sums gives the general kernels' bits, below either line it gives others."""
    import torch
    import paper_1412_6249_amd as pa
    from gpu_util import to_dev, workspace, to_host, rel_l2, DEV
    N, C, H, K, R = case
    g = torch.Generator().manual_seed(N + C)
    x, w, b = (torch.randn(s, generator=g) for s in ((N, C, H, H), (K, C, R, R), (K,)))
    desc, tx, tw, tb = pa.conv_desc(1, R // 2), x.to(DEV), w.to(DEV), b.to(DEV)

    def once():
        y = torch.full((N, K, H, H), float("nan"), device=DEV)
        pa.purine_conv_fwd_bias_relu(desc, tx, tw, tb, y, relu=True, ws=workspace(pa.purine_conv_workspace_bytes(0, desc, x.shape, w.shape, pa.PURINE_F32)))
        torch.cuda.synchronize()
        return y
    auto = once()
    _general(pa, True)
    try:
        general = once()
    finally:
        _general(pa, False)
    assert torch.equal(auto, general) == keeps
    assert rel_l2(to_host(auto), to_host(general)) <= 5e-6          # two fp32 sums of up to 2304 products each


def _huge_part(g, ref):
    """The outputs of 1e30 and more that are finite on both sides, scaled into range: (got, wanted)."""
    m = np.isfinite(g) & np.isfinite(ref) & (np.abs(ref) >= 1e30) & (np.abs(ref) < 3e38)
    return g[m].astype(np.float64) / 2.0 ** 100, ref[m] / 2.0 ** 100


@pytest.mark.parametrize("route", ["patch", "packets"])
def test_infinities_nans_and_values_at_the_upper_end_of_the_range(route):
    """An infinity times the zero low parts of the other operand is a NaN in the split products, and a value of 2^112
    and more has no scaled parts: outputs that come out infinite or NaN are computed again the way the fp32 kernel
    would. Same infinities, same NaNs as the general kernel; the finite ones right, small and huge."""
    import paper_1412_6249_amd as pa
    from gpu_util import rel_l2
    case = (2, 200, 12, 12, 208, 3, 3, 1, 1)
    x, w, b, dy, act, prev = _inputs(case)
    big = np.float32(3.4028234e38)
    x[0, 3, 2, 2], x[0, 5, 9, 9], x[1, 0, 0, 0], x[1, 7, 6, 6] = np.inf, np.nan, -np.inf, big
    x[1, 9, 3, 9] = 3e34                        # (above what the split holds, below the largest bf16)
    dy[0, 1, 3, 3], dy[1, 2, 8, 8], dy[1, 40, 1, 10] = -np.inf, np.nan, big
    w *= np.float32(0.1)                        # so that no finite partial sum overflows, whatever the order
    w[4, 4, 0, 0] = np.inf
    x[0, :, 5, 5] *= np.float32(1e-30)
    try:
        _forced(pa, route)
        got, _ = _run(pa, case, x, w, b, dy, act, prev)
        _forced(pa, "general")
        base, _ = _run(pa, case, x, w, b, dy, act, prev)
    finally:
        _forced(pa, "auto")
    assert not np.array_equal(got[1], base[1], equal_nan=True) and not np.array_equal(got[2], base[2], equal_nan=True)
    with np.errstate(all="ignore"):
        y, dx = oracle.conv_fwd(x, w, 1, 1), oracle.conv_bwd_data(dy, w, x.shape, 1, 1)
    for name, g, o, r in zip(("y fused", "y", "dx", "dx accumulated", "dx masked"), got, base, (None, y, dx, None, None)):
        assert np.array_equal(np.isnan(g), np.isnan(o)), name
        inf = np.isinf(o)
        assert np.array_equal(np.isinf(g), inf) and np.array_equal(g[inf], o[inf]), name
        ok = np.isfinite(o) & (np.abs(o) < 1e30)
        assert ok.mean() > 0.4 and rel_l2(g[ok], o[ok]) <= 1e-6, name
        if r is not None:                       # one fp32 sum that a single product dominates
            have, want = _huge_part(g, r)
            assert have.size > 500 and rel_l2(have, want) <= 1e-6 and (np.abs(have - want) <= 1e-5 * np.abs(want)).all(), name


# exponents of the small operand: where the third part of an unscaled split falls below the smallest bf16 (2^-133) in
# part and altogether, and where the second one does
@pytest.mark.parametrize("power", [-112, -117, -121])
@pytest.mark.parametrize("route", ["patch", "packets", "auto"])
def test_tiny_operands_keep_their_bits(route, power):
    """A whole operand close to the smallest normal number, the other one large: no less exact than the general kernels.
    (An operand held in two parts is off by 4e-6 at 2^-117, in one and a bit by 6e-5 at 2^-121.)"""
    import paper_1412_6249_amd as pa
    from gpu_util import rel_l2
    case = (8, 64, 14, 13, 72, 3, 3, 1, 1)
    tiny, large = np.float32(2.0 ** power), np.float32(2.0 ** 60)
    for small_filter in (False, True):
        x, w, b, dy, act, prev = _inputs(case)
        x, dy, w = (x * large, dy * large, w * tiny) if small_filter else (x * tiny, dy * tiny, w * large)
        b, prev = b * np.float32(0), prev * np.float32(0)
        got = {}
        try:
            for r in (route, "general"):
                _forced(pa, r)
                got[r], _ = _run(pa, case, x, w, b, dy, act, prev)
        finally:
            _forced(pa, "auto")
        y, dx = oracle.conv_fwd(x, w, 1, 1), oracle.conv_bwd_data(dy, w, x.shape, 1, 1)
        for name, g, o, ref in zip(("y", "dx"), got[route][1:3], got["general"][1:3], (y, dx)):
            assert np.abs(ref).max() > 0 and rel_l2(g, ref) <= max(rel_l2(o, ref), 1.0e-7), (name, small_filter, rel_l2(g, ref), rel_l2(o, ref))


@pytest.mark.parametrize("power", [-112, -117, -121])
def test_tiny_operands_keep_their_bits_in_the_weight_gradient_and_fc(power):
    import torch
    import paper_1412_6249_amd as pa
    from gpu_util import rel_l2, workspace
    case = (9, 48, 14, 13, 72, 3, 3, 1, 1)
    tiny, large = np.float32(2.0 ** power), np.float32(2.0 ** 60)
    for small_x in (False, True):
        x, w, b, dy, _, _ = _inputs(case)
        x, dy = (x * tiny, dy * large) if small_x else (x * large, dy * tiny)
        try:
            _forced(pa, "packets")
            got, _, _ = _wgrad(pa, case, x, dy, w, b, 0.0)
            _forced(pa, "general")
            base, _, _ = _wgrad(pa, case, x, dy, w, b, 0.0)
        finally:
            _forced(pa, "auto")
        ref = oracle.conv_bwd_weight(x, dy, w.shape, 1, 1)
        assert rel_l2(got, ref) <= max(rel_l2(base, ref), 1.0e-7), (small_x, rel_l2(got, ref), rel_l2(base, ref))
    N, C, K = 40, 2304, 2400                 # the weight gradient as a streaming product too
    g = torch.Generator().manual_seed(1)
    x, w, dy = (torch.randn(s, generator=g) for s in ((N, C), (K, C), (N, K)))
    err = lambda a, r: float((a.double().cpu() - r).norm() / r.norm())
    for a, c in ((float(tiny), float(large)), (float(large), float(tiny))):
        tx, tw, tdy = (x * a).cuda(), (w * c).cuda(), (dy * a).cuda()
        y, dx, dw = torch.empty(N, K, device="cuda"), torch.empty(N, C, device="cuda"), torch.empty(K, C, device="cuda")
        ws = [workspace(pa.purine_fc_workspace_bytes(p, N, C, K)) for p in (0, 1, 2)]
        pa.purine_fc_fwd(tx, tw, None, y, ws=ws[0])
        pa.purine_fc_bwd_data(tdy, tw, dx, ws=ws[1])
        pa.purine_fc_bwd_weight(tx, (dy * c).cuda(), dw, None, ws=ws[2])
        X, W, D, E = tx.double().cpu(), tw.double().cpu(), tdy.double().cpu(), (dy * c).double()
        # 2.5e-7 is the fp32 kernels' own error over sums of 2300; dw sums 40
        assert err(y, X @ W.t()) <= 3e-7 and err(dx, D @ W) <= 3e-7 and err(dw, E.t() @ X) <= 3e-7, (a, err(y, X @ W.t()), err(dx, D @ W), err(dw, E.t() @ X))


@pytest.mark.parametrize("route", ["patch", "packets"])
@pytest.mark.parametrize("amax", [2, 1000])
def test_integers_are_exact(amax, route):
    """Integers whose partial sums stay below 2^24 come out exactly, also those that need two parts."""
    import paper_1412_6249_amd as pa
    case = (2, 64, 8, 9, 72, 3, 3, 1, 1)
    rs = np.random.default_rng(3)
    x, w, b, dy, act, prev = (np.zeros_like(a) for a in _inputs(case))
    x[:] = rs.integers(-amax, amax + 1, x.shape)
    dy[:] = rs.integers(-amax, amax + 1, dy.shape)
    w[:] = rs.integers(-2, 3, w.shape)
    try:
        _forced(pa, route)
        got, _ = _run(pa, case, x, w, b, dy, act, prev)
    finally:
        _forced(pa, "auto")
    assert np.array_equal(got[1], oracle.conv_fwd(x, w, 1, 1).astype(np.float32))
    assert np.array_equal(got[2], oracle.conv_bwd_data(dy, w, x.shape, 1, 1).astype(np.float32))


# ---- weight gradient (conv_wgrad_packets.hip): eight images, or bands of eight images' rows, per packet
# N below, at and past a group of eight; odd planes (a padded position); bands with a ragged last one;
# channel counts around the 16-channel tiles of the layout pass; strides, unequal sides, columns past a tile
WCASES = [(8, 32, 9, 9, 48, 3, 3, 1, 1), (1, 16, 7, 5, 17, 3, 3, 1, 1), (5, 40, 9, 9, 24, 1, 1, 1, 0), (2, 3, 31, 29, 20, 7, 7, 2, 3), (1, 64, 16, 14, 96, 3, 3, 1, 1), (3, 70, 13, 11, 33, 3, 3, 1, 1), (2, 33, 24, 17, 40, 5, 3, 1, (2, 1)),
          (17, 40, 12, 13, 65, 3, 3, 2, 1), (12, 72, 31, 30, 130, 5, 4, (3, 2), (2, 1)), (9, 130, 8, 8, 70, 2, 2, 1, 0), (29, 41, 25, 19, 95, 3, 5, 1, (0, 2))]


def _wgrad(pa, case, x, dy, prev_w, prev_b, beta):
    import torch
    from gpu_util import to_dev, workspace, to_host
    desc = pa.conv_desc(case[7], case[8])
    need = pa.purine_conv_workspace_bytes(pa.PURINE_CONV_BWD_WEIGHT_BIAS, desc, x.shape, prev_w.shape, pa.PURINE_F32)
    tx, tdy, dw, db, alone = to_dev(x), to_dev(dy), to_dev(prev_w), to_dev(prev_b), to_dev(prev_w)
    ws = workspace(need)
    ws.fill_(0xff)                   # NaN patterns: nothing may be read that was not written
    pa.purine_conv_bwd_weight_bias(desc, tx, tdy, dw, db, beta=beta, ws=ws)
    ws.fill_(0xff)
    pa.purine_conv_bwd_weight(desc, tx, tdy, alone, beta=beta, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(dw.view(torch.int32), alone.view(torch.int32))       # the same bits (NaNs too)
    return to_host(dw), to_host(db), need


@pytest.mark.parametrize("beta", [0.0, 1.0])
@pytest.mark.parametrize("case", WCASES, ids=str)
def test_weight_gradient_on_packed_parts(case, beta):
    import paper_1412_6249_amd as pa
    from gpu_util import rel_l2
    x, w, b, dy, _, _ = _inputs(case)
    try:
        _forced(pa, "packets")
        got_w, got_b, need = _wgrad(pa, case, x, dy, w, b, beta)
        _forced(pa, "general")
        base_w, _, need0 = _wgrad(pa, case, x, dy, w, b, beta)
    finally:
        _forced(pa, "auto")
    assert need != need0                 # the layer takes the packed kernel: its scratch holds the packed operands
    ref = oracle.conv_bwd_weight(x, dy, w.shape, case[7], case[8]) + beta * w
    ref_b = oracle.bias_bwd(dy) + beta * b
    # the result's own rounding is 0.3 * 2^-24; the sums beyond it may be no further off than the general kernel's
    assert rel_l2(got_w, ref) <= max(rel_l2(base_w, ref), 1.0e-7), (rel_l2(got_w, ref), rel_l2(base_w, ref))
    assert rel_l2(got_b, ref_b) <= 1e-6


def test_weight_gradient_route_and_nonfinite_values():
    """The layer takes the packed kernel (its scratch holds the packed operands), and infinities and NaNs
    come out where the general kernel has them: also next to padding, in the last band's missing rows and
    in the images a partial group lacks, where the other operand's zeros must not meet them."""
    import paper_1412_6249_amd as pa
    from gpu_util import rel_l2
    case = (5, 160, 15, 15, 192, 3, 3, 1, 1)
    x, w, b, dy, _, _ = _inputs(case)
    x[0, 3, 0, 0], x[4, 9, 14, 14], x[2, 20, 7, 7] = np.inf, -np.inf, np.nan
    x[1, 30, 3, 3] = np.float32(3.4028234e38)
    dy *= np.float32(1e-3)
    dy[4, 5, 14, 14], dy[3, 8, 0, 7], dy[0, 63, 10, 10] = np.inf, np.nan, -np.inf
    x[1, 31, 5, 5], dy[1, 100, 6, 6] = 1e34, np.float32(2e36)
    got_w, got_b, need = _wgrad(pa, case, x, dy, w, b, 0.0)
    _general(pa, True)
    try:
        base_w, base_b, need0 = _wgrad(pa, case, x, dy, w, b, 0.0)
    finally:
        _general(pa, False)
    assert need != need0
    with np.errstate(all="ignore"):
        have, want = _huge_part(got_w, oracle.conv_bwd_weight(x, dy, w.shape, 1, 1))
    # several products of that size may cancel: the bound on a sum's terms instead of on the sum
    assert have.size > 500 and rel_l2(have, want) <= 1e-5
    for g, o in ((got_w, base_w), (got_b, base_b)):
        assert np.array_equal(np.isnan(g), np.isnan(o))
        inf = np.isinf(o)
        assert np.array_equal(np.isinf(g), inf) and np.array_equal(g[inf], o[inf])
        ok = np.isfinite(o) & (np.abs(o) < 1e30)
        assert ok.any() and rel_l2(g[ok], o[ok]) <= 1e-6


def test_weight_gradient_in_the_static_scratch_takes_the_splits_in_turn():
    """The packed operands of this layer do not fit the static scratch at once; the entry point packs and
    multiplies a few splits at a time and gives the same bits as the call with a workspace."""
    import torch
    import paper_1412_6249_amd as pa
    from gpu_util import workspace, rel_l2, to_host, DEV
    N, C, H, W, K = 24, 128, 56, 56, 128
    g = torch.Generator(device=DEV)
    g.manual_seed(7)
    x = torch.randn((N, C, H, W), generator=g, device=DEV)
    dy = torch.randn((N, K, H, W), generator=g, device=DEV)
    desc = pa.conv_desc(1, 1)
    need = pa.purine_conv_workspace_bytes(pa.PURINE_CONV_BWD_WEIGHT, desc, x.shape, (K, C, 3, 3), pa.PURINE_F32)
    assert need > pa.purine_static_scratch_bytes()
    want, got, base = (torch.full((K, C, 3, 3), float("nan"), device=DEV) for _ in range(3))
    pa.purine_conv_bwd_weight(desc, x, dy, want, ws=workspace(need))
    for _ in range(2):
        pa.purine_conv_bwd_weight_static(desc, x, dy, got)
    _general(pa, True)
    try:
        pa.purine_conv_bwd_weight_static(desc, x, dy, base)
    finally:
        _general(pa, False)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    assert rel_l2(to_host(got), to_host(base)) <= 2e-6        # two fp32 sums of 75264 products each


def _time_of(f, calls=30):
    """Least time of one call over a few rounds of `calls`, in seconds."""
    import time
    import torch
    best = float("inf")
    for _ in range(6):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(calls):
            f()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / calls)
    return best


# few images of a first layer: three channels, many taps, many splits of the pixel reduction
@pytest.mark.parametrize("case", [(4, 3, 100, 102, 55, 11, 11, 2, 5), (23, 3, 68, 70, 107, 11, 11, 4, 0), (7, 3, 184, 185, 124, 7, 7, 4, 3),
                                  (1, 16, 38, 38, 56, 3, 3, 1, 0), (2, 8, 20, 20, 176, 5, 5, 1, 2)], ids=str)
def test_weight_gradient_takes_no_longer_than_on_the_general_kernel(case):
    """The automatic route against the general kernels over the same layer. A quarter more is what these calls of
    15 - 40 us vary by; the second pass that walked taps times splits one by one took 2 - 8 times as long."""
    import paper_1412_6249_amd as pa
    from gpu_util import to_dev, workspace
    x, w, b, dy, _, _ = _inputs(case)
    desc, tx, tdy, dw, db = pa.conv_desc(case[7], case[8]), to_dev(x), to_dev(dy), to_dev(w), to_dev(b)

    def once():
        ws = workspace(pa.purine_conv_workspace_bytes(pa.PURINE_CONV_BWD_WEIGHT_BIAS, desc, x.shape, w.shape, pa.PURINE_F32))
        return _time_of(lambda: pa.purine_conv_bwd_weight_bias(desc, tx, tdy, dw, db, ws=ws))
    auto = once()
    _general(pa, True)
    try:
        general = once()
    finally:
        _general(pa, False)
    assert auto <= 1.25 * general, (auto, general)


# N, C, K of a fully-connected layer: rows and columns one past a tile, reductions that are no whole step (and no
# whole 16-byte packet), reductions split over workgroups, batches on either side of the weight gradient's rule,
# operands laid out first (dw of the wide ones)
FC_CASES = [(1, 4, 4), (33, 129, 65), (32, 130, 1001), (129, 1023, 257), (65, 2049, 1000), (40, 1026, 1030), (97, 640, 33), (128, 3000, 4100)]


@pytest.mark.parametrize("case", FC_CASES)
def test_fc_f32(case):
    """The three passes against fp64, no less exact than the general kernels; twice the same bits; onto a previous
    gradient; whole numbers exactly; infinities and NaN as a plain sum has them."""
    import torch
    import paper_1412_6249_amd as pa
    from gpu_util import workspace
    N, C, K = case
    g = torch.Generator().manual_seed(N + C)
    f = lambda *s: torch.randn(*s, generator=g)
    x, w, b, dy, prev = f(N, C), f(K, C), f(K), f(N, K), f(K, C)

    def run(x, w, b, dy, prev):
        x, w, b, dy, acc = (t.cuda() for t in (x, w, b, dy, prev))
        nan = lambda *s: torch.full(s, float("nan"), device="cuda")
        ws = [workspace(pa.purine_fc_workspace_bytes(p, N, C, K)) for p in (0, 1, 2)]
        y, dx, dw, db = nan(N, K), nan(N, C), nan(K, C), nan(K)
        pa.purine_fc_fwd(x, w, b, y, ws=ws[0])
        pa.purine_fc_bwd_data(dy, w, dx, ws=ws[1])
        pa.purine_fc_bwd_weight(x, dy, dw, db, ws=ws[2])
        pa.purine_fc_bwd_weight(x, dy, acc, None, beta=1.0, ws=ws[2])
        torch.cuda.synchronize()
        return [t.cpu() for t in (y, dx, dw, db, acc)]

    def want(x, w, b, dy, prev):
        x, w, b, dy, prev = (t.double() for t in (x, w, b, dy, prev))
        return [x @ w.t() + b, dy @ w, dy.t() @ x, dy.sum(0), dy.t() @ x + prev]

    err = lambda got, ref: [float((a.double() - r).norm() / r.norm()) for a, r in zip(got, ref)]
    got, again, ref = run(x, w, b, dy, prev), run(x, w, b, dy, prev), want(x, w, b, dy, prev)
    assert all(torch.equal(a, c) for a, c in zip(got, again))
    _general(pa, True)
    try:
        plain = run(x, w, b, dy, prev)
    finally:
        _general(pa, False)
    # 2^-24 per output is one rounding of the result, which either may have more of
    assert all(e <= p + 2.0 ** -24 for e, p in zip(err(got, ref), err(plain, ref))), (err(got, ref), err(plain, ref))

    ints = [t.mul(3).round() for t in (x, w, b, dy, prev)]       # sums far below 2^24: exact in any order
    assert all(torch.equal(a.double(), r) for a, r in zip(run(*ints), want(*ints)))

    bad = [t.clone() for t in (x, w, b, dy, prev)]
    bad[0][N // 2, C - 1], bad[1][K - 1, 0], bad[3][0, K - 1] = float("inf"), float("nan"), float("-inf")
    for a, r in zip(run(*bad), want(*bad)):
        assert torch.equal(a.isnan(), r.isnan()) and torch.equal(a.isposinf(), r.isposinf()) and torch.equal(a.isneginf(), r.isneginf())


def _graph_time_of(f, calls=20):
    """Least time of one call among `calls` captured into a graph, in seconds: the GPU's alone."""
    import time
    import torch
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        f()
        st.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            for _ in range(calls):
                f()
        best = float("inf")
        for _ in range(6):
            st.synchronize()
            t = time.perf_counter()
            g.replay()
            st.synchronize()
            best = min(best, (time.perf_counter() - t) / calls)
    return best


# dw on 128-row tiles that spilled their accumulators; dx of a batch one past a tile on 96-row ones; sums of one
# step; a short weight gradient whose batch is no whole step
@pytest.mark.parametrize("which, case", [("dw", (48, 3140, 1780)), ("dw", (231, 1000, 200)), ("dw", (200, 9000, 64)),
                                         ("dx", (131, 9216, 4096)), ("dx", (100, 256, 10)), ("dx", (128, 169, 247))])
def test_fc_f32_takes_no_longer_than_the_composition(which, case):
    """The automatic route against the composition of convolution kernels. A quarter more is allowed; these calls took
    1.3 - 3 times as long before the route weighed both."""
    import torch
    import paper_1412_6249_amd as pa
    from gpu_util import workspace
    N, C, K = case
    x, w, dy = (torch.randn(s, device="cuda") for s in ((N, C), (K, C), (N, K)))
    out = torch.empty_like(w if which == "dw" else x)

    def once():
        ws = workspace(pa.purine_fc_workspace_bytes(pa.PURINE_CONV_BWD_WEIGHT if which == "dw" else pa.PURINE_CONV_BWD_DATA, N, C, K))
        if which == "dw":
            return _graph_time_of(lambda: pa.purine_fc_bwd_weight(x, dy, out, None, ws=ws))
        return _graph_time_of(lambda: pa.purine_fc_bwd_data(dy, w, out, ws=ws))
    auto = once()
    _general(pa, True)
    try:
        general = once()
    finally:
        _general(pa, False)
    assert auto <= 1.25 * general, (auto, general)


@pytest.mark.parametrize("which, N, H, stride", [("forward", 64, 56, 2), ("weight gradient", 128, 28, 1)])
def test_timing_bracket_holds_the_layout_pass(which, N, H, stride):
    """A pass that lays its operands out first is bracketed from there to its second pass: what the bracket reads is
    what a call takes on the device (the products alone are about two thirds of these)."""
    import torch
    import paper_1412_6249_amd as pa
    from gpu_util import workspace, DEV
    C, K, P = 96, 128, H // stride
    desc = pa.conv_desc(stride, 1)
    x, w, dy = (torch.randn(s, device=DEV) for s in ((N, C, H, H), (K, C, 3, 3), (N, K, P, P)))
    y, dw = torch.empty_like(dy), torch.empty_like(w)
    p = pa.PURINE_CONV_FWD if which == "forward" else pa.PURINE_CONV_BWD_WEIGHT
    assert pa.purine_conv_matrix_products(p, desc, x.shape, w.shape, pa.PURINE_F32) == 6
    ws = workspace(pa.purine_conv_workspace_bytes(p, desc, x.shape, w.shape, pa.PURINE_F32))
    f = (lambda: pa.purine_conv_fwd(desc, x, w, y, ws=ws)) if which == "forward" else (lambda: pa.purine_conv_bwd_weight(desc, x, dy, dw, ws=ws))
    whole = _graph_time_of(f)
    evs = [[torch.cuda.Event(enable_timing=True) for _ in range(2)] for _ in range(20)]
    for s, e in evs:                       # create the underlying handles
        s.record(); e.record()
    torch.cuda.synchronize()
    for s, e in evs:
        pa.purine_set_kernel_probe(s.cuda_event, e.cuda_event)
        f()
    pa.purine_set_kernel_probe(None, None)
    torch.cuda.synchronize()
    bracket = min(s.elapsed_time(e) for s, e in evs) * 1e-3
    assert 0.9 * whole <= bracket <= 1.3 * whole + 1e-5, (bracket, whole)
