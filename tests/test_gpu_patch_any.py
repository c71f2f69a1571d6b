"""The bf16 patch kernel for rows of any width: every tile and both request schemes at the edges of tiles, channel
groups, rows and images, against the oracle, and bit for bit against each other (all of them add a channel
group's taps in the same order). The tensors are channel slices whose neighbours hold NaN: what a kernel reads past a
slice's last channel must not reach a result."""
import numpy as np
import pytest

import oracle
from synth import gen

gpu = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad. The smallest width and patch, odd planes (every other channel at an odd element), last
# loads that overlap, one row past a tile, channels on either side of a group of 16 and of 8, many images per tile, filters
# with a kernel of their own (2x2 folded, 3x3, 5x5) and without, strides that gather and that fold, rows wider than a tile
CASES = [(2, 16, 4, 4, 33, 3, 3, 1, 1), (3, 17, 7, 7, 32, 3, 3, 1, 1), (70, 24, 5, 5, 16, 3, 3, 1, 0), (2, 31, 13, 13, 97, 3, 3, 1, 1),
         (1, 33, 28, 28, 129, 3, 3, 1, 1), (2, 40, 14, 9, 20, 5, 5, 1, 2), (3, 16, 11, 13, 40, 3, 3, 2, 1), (2, 24, 12, 15, 33, 5, 5, 2, 2),
         (2, 19, 10, 11, 24, 2, 3, 1, (1, 0)), (1, 48, 9, 17, 17, 1, 5, 1, (0, 2)), (2, 16, 14, 19, 30, 4, 4, (3, 2), (2, 1)),
         (2, 20, 6, 131, 18, 3, 3, 1, 1), (1, 64, 33, 37, 65, 3, 3, 1, 1), (4, 23, 9, 8, 41, 3, 2, (1, 2), (1, 0))]
TILES = (128256, 96256, 96128, 64256, 64128, 32256, 32128, 1032128)
AUTO, FAR = 0, -1              # the plan's own tile; the same with the addresses of tensors of 2^31 bytes and more


def _filter_bytes(case, which, bm):
    """Scratch of a pass on this kernel with row tiles of bm, its filter copy: no other kernel for these layers asks for as little."""
    N, C, H, W, K, R, S, stride, pad = case
    sh, sw = stride if isinstance(stride, tuple) else (stride, stride)
    if which == 0 or (sh, sw) == (1, 1):
        rows, ch, taps = (K, C, R * S) if which == 0 else (C, K, R * S)
    else:
        rows, ch, taps = C * sh * sw, K, -(-R // sh) * -(-S // sw)
    return -(-rows // bm) * bm * -(-ch // 16) * 16 * taps * 2


def _taken(case, which, tile):
    """Whether the pass runs on this kernel with the forced tile."""
    import paper_1412_6249_amd as pa
    N, C, H, W, K, R, S, stride, pad = case
    pa.purine_debug_force_tile(-9, tile)
    try:
        need = pa.purine_conv_workspace_bytes(which, pa.conv_desc(stride, pad), (N, C, H, W), (K, C, R, S), pa.PURINE_BF16)
    finally:
        pa.purine_debug_force_tile(0, 0)
    return need in {_filter_bytes(case, which, bm) for bm in ([tile % 1000000 // 1000] if tile > 0 else (32, 64, 96, 128))}


def test_every_tile_is_taken():
    """Passes of CASES on each tile: forward, backward-data, folded backward-data among them. (The third layer's gradient has
    rows of three pixels; depth-to-space has no 128x256 and 96x256 tile; the last needs a filter with a kernel of its own.)"""
    for tile in (AUTO, FAR) + TILES:
        got = [sum(_taken(c, which, tile) for c in CASES if folded is None or c[7] != 1) for which, folded in ((0, None), (1, None), (1, True))]
        want = {128256: (13, 9, 0), 96256: (13, 9, 0), 1032128: (7, 9, 3)}.get(tile, (13, 13, 4))
        assert all(g >= w for g, w in zip(got, want)), (tile, got)


def _slice(a, lead, tail):
    """The values of `a` as the middle channels of a tensor that holds NaN everywhere else."""
    import torch
    from gpu_util import to_dev, DEV
    n, c, h, w = a.shape
    big = torch.full((n, c + lead + tail, h, w), float("nan"), dtype=torch.bfloat16, device=DEV)
    view = big[:, lead:lead + c]
    view.copy_(to_dev(a, "bf16"))
    return view


@gpu
@pytest.mark.parametrize("case", CASES, ids=str)
def test_every_tile_against_the_oracle(case):
    import torch
    import paper_1412_6249_amd as pa
    from gpu_util import rel_l2, to_dev, to_host, workspace, TOL
    N, C, H, W, K, R, S, stride, pad = case
    rs = np.random.default_rng(3)
    f = lambda *s: gen.quantize_bf16(rs.uniform(-1, 1, s).astype(np.float32))
    P, Q = oracle.out_shape((N, C, H, W), (K, C, R, S), stride, pad)[2:]
    x, w, b, dy, act, prev = f(N, C, H, W), f(K, C, R, S), f(K), f(N, K, P, Q), f(N, C, H, W), f(N, C, H, W)
    y = np.maximum(oracle.bias_fwd(oracle.conv_fwd(x, w, stride, pad), b), 0)
    dx = oracle.conv_bwd_data(dy, w, x.shape, stride, pad)
    refs = (y, dx, dx + prev, np.where(act > 0, dx, 0.0))
    desc, first = pa.conv_desc(stride, pad), None
    # slices start at whole 16-byte packets
    pad_x, pad_y = (8 if H * W % 8 else 1), (8 if P * Q % 8 else 1)
    up = lambda c, m: c + (-c) % m
    for tile in (AUTO, FAR) + TILES:
        # (a forced tile that does not apply leaves the call on another kernel)
        taken = [_taken(case, which, tile) for which in (0, 1, 1, 1)]
        pa.purine_debug_force_tile(-9, tile)
        try:
            tx, tdy, tact = _slice(x, pad_x, up(C, pad_x) - C), _slice(dy, pad_y, up(K, pad_y) - K), _slice(act, pad_x, up(C, pad_x) - C)
            ty = _slice(np.zeros_like(dy), pad_y, up(K, pad_y) - K)
            td, ta, tm = (_slice(v, pad_x, up(C, pad_x) - C) for v in (np.zeros_like(x), prev, np.zeros_like(x)))
            tw, tb = to_dev(w, "bf16"), to_dev(b, "bf16")
            ws = [workspace(pa.purine_conv_workspace_bytes(k, desc, x.shape, w.shape, pa.PURINE_BF16)) for k in (0, 1)]
            pa.purine_conv_fwd_bias_relu(desc, tx, tw, tb, ty, relu=True, ws=ws[0])
            pa.purine_conv_bwd_data(desc, tdy, tw, td, ws=ws[1])
            pa.purine_conv_bwd_data(desc, tdy, tw, ta, beta=1.0, ws=ws[1])
            pa.purine_conv_bwd_data_relu(desc, tdy, tw, tact, tm, ws=ws[1])
            torch.cuda.synchronize()
        finally:
            pa.purine_debug_force_tile(0, 0)
        got = [to_host(t) for t in (ty, td, ta, tm)]
        for name, g, r in zip(("y", "dx", "dx accumulated", "dx masked"), got, refs):
            assert rel_l2(g, r) <= TOL["bf16"], (tile, name, rel_l2(g, r))
        if first is None:
            first = got
        for name, g, r, same in zip(("y", "dx", "dx accumulated", "dx masked"), got, first, taken):
            assert not same or np.array_equal(g, r), (tile, name)
        for t, ch in ((ty, K), (td, C), (ta, C), (tm, C)):
            assert int(torch.isnan(t._base).sum()) == t._base.numel() - t.numel(), "stored outside the slice"


# N, C, H, W, K, R, S, stride, pad: filters with a kernel of their own, whose requests run a group or several ahead, and without
FAR_CASES = [(3, 24, 17, 19, 40, 3, 3, 1, 1), (3, 40, 14, 16, 97, 5, 5, 1, 2), (3, 17, 9, 8, 16, 3, 2, 1, (1, 0)), (3, 33, 28, 28, 130, 3, 3, 2, 1)]


@gpu
@pytest.mark.parametrize("case", FAR_CASES, ids=str)
def test_images_far_apart(case):
    """x, y and their gradients as slices whose images lie up to 4 GB apart (spans of almost 2^31 elements, past 2^31 bytes, which
    no raw buffer addresses): the same bits as from dense tensors, with the scratch of the one query there is."""
    import torch
    import paper_1412_6249_amd as pa
    from gpu_util import to_dev, workspace, DEV
    N, C, H, W, K, R, S, stride, pad = case
    P, Q = oracle.out_shape((N, C, H, W), (K, C, R, S), stride, pad)[2:]
    rs = np.random.default_rng(5)
    f = lambda *s: to_dev(gen.quantize_bf16(rs.uniform(-1, 1, s).astype(np.float32)), "bf16")
    x, w, b, dy, act, prev = f(N, C, H, W), f(K, C, R, S), f(K), f(N, K, P, Q), f(N, C, H, W), f(N, C, H, W)
    desc = pa.conv_desc(stride, pad)
    ws = [workspace(pa.purine_conv_workspace_bytes(k, desc, x.shape, w.shape, pa.PURINE_BF16)) for k in (0, 1)]
    flat = [torch.empty(2 ** 31, dtype=torch.bfloat16, device=DEV) for _ in range(3)]

    def far(i, t):
        ns = (2 ** 31 - t[0].numel() - 1) // (N - 1) // 8 * 8
        return flat[i].as_strided(t.shape, (ns,) + t.stride()[1:]).copy_(t)

    def run(x, dy, act, out_y, out_dx):
        y, dx = out_y(torch.zeros_like(dy)), out_dx(torch.zeros_like(x))
        got = []
        for relu in (True, False):
            pa.purine_conv_fwd_bias_relu(desc, x, w, b, y, relu=relu, ws=ws[0])
            got.append(y.clone())
        pa.purine_conv_bwd_data(desc, dy, w, dx, ws=ws[1])
        got.append(dx.clone())
        dx.copy_(prev)
        pa.purine_conv_bwd_data(desc, dy, w, dx, beta=1.0, ws=ws[1])
        got.append(dx.clone())
        pa.purine_conv_bwd_data_relu(desc, dy, w, act, dx, ws=ws[1])
        got.append(dx.clone())
        torch.cuda.synchronize()
        return [t.contiguous() for t in got]

    same = lambda t: t
    want = run(x, dy, act, same, same)
    # far inputs, dense outputs; then far outputs (the ReLU mask has dx's strides)
    got_in = run(far(0, x), far(1, dy), act, same, same)
    got_out = run(x, dy, far(1, act), lambda t: far(0, t), lambda t: far(2, t))
    for name, g, h, r in zip(("relu(y + b)", "y + b", "dx", "dx accumulated", "dx masked"), got_in, got_out, want):
        assert torch.equal(g, r) and torch.equal(h, r), name


# rows of whole packets too wide for this kernel's patch, both ways: the one-image kernel (two fill rounds), strided backward too
WIDE_CASES = [(2, 16, 5, 264, 24, 3, 3, 1, 1), (1, 24, 7, 1056, 16, 3, 3, 2, 1)]


@gpu
@pytest.mark.parametrize("case", WIDE_CASES, ids=str)
def test_rows_too_wide_for_a_patch(case):
    import torch
    import paper_1412_6249_amd as pa
    from gpu_util import rel_l2, to_dev, to_host, workspace, TOL
    N, C, H, W, K, R, S, stride, pad = case
    rs = np.random.default_rng(1)
    f = lambda *s: gen.quantize_bf16(rs.uniform(-1, 1, s).astype(np.float32))
    P, Q = oracle.out_shape((N, C, H, W), (K, C, R, S), stride, pad)[2:]
    x, w, b, dy, act, prev = f(N, C, H, W), f(K, C, R, S), f(K), f(N, K, P, Q), f(N, C, H, W), f(N, C, H, W)
    desc = pa.conv_desc(stride, pad)
    need = [pa.purine_conv_workspace_bytes(k, desc, x.shape, w.shape, pa.PURINE_BF16) for k in (0, 1)]
    one_image = [k for k in (0, 1) if need[k] == max(_filter_bytes(case, k, 96), _filter_bytes(case, k, 128))]
    assert one_image == ([0, 1] if stride == 1 else [1])        # (a strided forward gather takes the blocked copy)
    ws = [workspace(n) for n in need]
    d = lambda a: to_dev(a, "bf16")
    tx, tw, tb, tdy, tact = d(x), d(w), d(b), d(dy), d(act)
    y, relu_y = torch.zeros_like(tdy), torch.zeros_like(tdy)
    dx, dxa, dxm = torch.zeros_like(tx), d(prev), torch.zeros_like(tx)
    pa.purine_conv_fwd_bias_relu(desc, tx, tw, tb, y, relu=False, ws=ws[0])
    pa.purine_conv_fwd_bias_relu(desc, tx, tw, tb, relu_y, relu=True, ws=ws[0])
    pa.purine_conv_bwd_data(desc, tdy, tw, dx, ws=ws[1])
    pa.purine_conv_bwd_data(desc, tdy, tw, dxa, beta=1.0, ws=ws[1])
    pa.purine_conv_bwd_data_relu(desc, tdy, tw, tact, dxm, ws=ws[1])
    torch.cuda.synchronize()
    ref_y = oracle.bias_fwd(oracle.conv_fwd(x, w, stride, pad), b)
    ref = oracle.conv_bwd_data(dy, w, x.shape, stride, pad)
    for name, g, r in (("y", y, ref_y), ("relu(y)", relu_y, np.maximum(ref_y, 0)), ("dx", dx, ref), ("dx accumulated", dxa, ref + prev),
                       ("dx masked", dxm, np.where(act > 0, ref, 0.0))):
        assert rel_l2(to_host(g), r) <= TOL["bf16"], name
