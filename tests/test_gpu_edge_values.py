"""Edges of the small passes and of the products: infinities in the operands of the expert products, segments longer than
the window of the token-dropping pass, the merged pass over the combine weights' gradient, routing over NaNs, the bits of the
float32 products, tile maps of many experts.

Integers, copies and what an infinity does not reach are compared bit for bit; the many-experts products as in
test_gpu_direct_tiles.py's reasoning for float32: sums of at most 64 terms of order one, 2^-24 each, held to 2^-16."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import check_capped_eri, i32, run_build_eri

pytestmark = pytest.mark.gpu


def gathered_rows(a):
    """(token matrix, row index) that stand for the rows of a."""
    p = torch.randperm(a.shape[0], generator=torch.Generator().manual_seed(a.shape[0]))
    t = torch.empty_like(a)
    t[p] = a
    return t.cuda(), p.int().cuda()


def ffn(m, rows, x, w, dy, gu=None, gathered=False):
    """Forward and backward of one call (gu: the backward starts from these instead; gathered: rows of x and dy through an
    index): name -> host tensor."""
    off = torch.tensor([0] + list(torch.tensor(rows).cumsum(0)), dtype=torch.int32).cuda()
    (B, d), (E, _, f), dt = x.shape, w[0].shape, x.dtype
    new = lambda *s: torch.empty(s, dtype=dt, device="cuda")
    o = {"g": new(B, f), "u": new(B, f), "y": new(B, d), "dxd": new(B, d), "dwg": new(E, d, f), "dwu": new(E, d, f),
         "dwd": new(E, f, d)}
    code = m.XMOE_F32 if dt == torch.float32 else m.XMOE_BF16
    ws = m.alloc_workspace(max(m.xmoe_workspace_bytes(op, B, d, E, 1, f, code) for op in (m.WS_FFN_FWD, m.WS_FFN_BWD)))
    (xc, xi), (dc, di) = (gathered_rows(a) if gathered else (a.cuda(), None) for a in (x, dy))
    wc = [a.cuda() for a in w]
    m.xmoe_expert_ffn_fwd(xc, off, *wc, o["g"], o["u"], o["y"], ws, row_index=xi)
    g, u = (o["g"], o["u"]) if gu is None else (t.cuda() for t in gu)
    m.xmoe_expert_ffn_bwd(xc, g, u, dc, off, *wc, o["dxd"], o["dwg"], o["dwu"], o["dwd"], ws, row_index=xi, dy_row_index=di)
    return {n: t.float().cpu() for n, t in o.items()}


def random_ffn(rows, d, f, dt):
    g = torch.Generator().manual_seed(d + f)
    E, B = len(rows), sum(rows)
    r = lambda *s: torch.randn(s, generator=g).to(dt)
    return r(B, d), [r(E, d, f) * d ** -0.5, r(E, d, f) * d ** -0.5, r(E, f, d) * f ** -0.5], r(B, d)


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("gathered", [False, True])
@pytest.mark.parametrize("rows,d,f", [([70, 5, 130], 72, 40), ([70, 5, 130], 33, 129), ([0, 300, 260, 1] * 8, 328, 264),
                                      ([0, 3000, 5200, 1], 520, 500)])   # the last: 128 x 128 tiles of every product
def test_infinities_go_where_the_products_take_them(rows, d, f, dt, gathered):
    import functools
    import paper_2508_13337_amd as m
    ffn = functools.partial(globals()["ffn"], gathered=gathered)
    x, w, dy = random_ffn(rows, d, f, dt)
    e = 2 if rows[0] else 1
    lo, hi = sum(rows[:e]), sum(rows[:e + 1])
    r, kd, kf = lo + 2, d - 1, f - 1
    clean = ffn(m, rows, x, w, dy)
    inf = float("inf")

    def same_outside(name, got, mask):
        assert torch.equal(got[name][~mask], clean[name][~mask]), name

    # a row of x: its row of G and U is infinite with the weights' signs, no other row changes
    x1 = x.clone()
    x1[r, kd] = inf
    o = ffn(m, rows, x1, w, dy)
    for name, a in (("g", w[0]), ("u", w[1])):
        assert torch.equal(o[name][r], inf * a[e, kd].float().sign()), name
    for name in ("g", "u", "y", "dxd"):
        mask = torch.zeros_like(o[name], dtype=torch.bool)
        mask[r] = True
        same_outside(name, o, mask)
    # a weight of Wd: its column of the expert's Y, with the activations' signs (A = silu(G) U has the sign of G U)
    w1 = [a.clone() for a in w]
    w1[2][e, kf, kd] = inf
    o = ffn(m, rows, x, w1, dy)
    sign = (clean["g"][lo:hi, kf].sign() * clean["u"][lo:hi, kf].sign())
    assert torch.equal(o["y"][lo:hi, kd], inf * sign)
    mask = torch.zeros_like(o["y"], dtype=torch.bool)
    mask[lo:hi, kd] = True
    same_outside("y", o, mask)
    # a row of dY: its column of dWd, with the activations' signs; no other expert's weight gradients change
    dy1 = dy.clone()
    dy1[r, kd] = inf
    o = ffn(m, rows, x, w, dy1)
    assert torch.equal(o["dwd"][e][:, kd], inf * clean["g"][r].sign() * clean["u"][r].sign())
    mask = torch.zeros_like(o["dwd"], dtype=torch.bool)
    mask[e, :, kd] = True
    same_outside("dwd", o, mask)
    for name in ("dwg", "dwu"):
        assert torch.equal(o[name][[i for i in range(len(rows)) if i != e]],
                           clean[name][[i for i in range(len(rows)) if i != e]]), name
    # a weight of Wu in the backward alone: its row's column of dXd is infinite
    w1 = [a.clone() for a in w]
    w1[1][e, kd, kf] = inf
    g, u = (clean[n].to(dt) for n in ("g", "u"))
    base, o = ffn(m, rows, x, w, dy, (g, u)), ffn(m, rows, x, w1, dy, (g, u))
    assert bool(torch.isinf(o["dxd"][lo:hi, kd]).all())
    mask = torch.zeros_like(o["dxd"], dtype=torch.bool)
    mask[lo:hi, kd] = True
    assert torch.equal(o["dxd"][~mask], base["dxd"][~mask])


@pytest.mark.parametrize("gathered", [False, True])
@pytest.mark.parametrize("act", ["identity", "silu"])
@pytest.mark.parametrize("rows,d,f", [([70, 5, 130], 72, 41), ([0, 3000, 5200, 1], 520, 500)])
def test_infinities_in_the_two_matrix_expert(rows, d, f, act, gathered):
    import paper_2508_13337_amd as m
    x, (w1, _, w2), dy = random_ffn(rows, d, f, torch.float32)
    off = torch.tensor([0] + list(torch.tensor(rows).cumsum(0)), dtype=torch.int32).cuda()
    E, B, r, e, inf = len(rows), sum(rows), sum(rows[:2]) + 2, 2, float("inf")
    x1, v2 = x.clone(), w2.clone()
    x1[r, d - 1] = inf
    v2[e, f - 1, 3] = inf
    outs = []
    for xs, ws2 in ((x, w2), (x1, w2), (x, v2)):
        new = lambda *s: torch.empty(s, device="cuda")
        o = {"h": new(B, f), "y": new(B, d), "dxd": new(B, d), "dw1": new(E, d, f), "dw2": new(E, f, d)}
        (xc, xi), (dc, di) = (gathered_rows(a) if gathered else (a.cuda(), None) for a in (xs, dy))
        ws = m.alloc_workspace(max(m.xmoe_workspace_bytes(op, B, d, E, 1, f, m.XMOE_F32) for op in (m.WS_MLP2_FWD, m.WS_MLP2_BWD)))
        wc = w1.cuda(), ws2.cuda()
        m.xmoe_expert_mlp2_fwd(xc, off, *wc, act, o["h"], o["y"], ws, row_index=xi)
        m.xmoe_expert_mlp2_bwd(xc, o["h"], dc, off, *wc, act, o["dxd"], o["dw1"], o["dw2"], ws, row_index=xi, dy_row_index=di)
        outs.append({n: t.cpu() for n, t in o.items()})
    clean, row, weight = outs
    # a row of x: its row of H, with the weights' signs, and no other row of anything
    assert torch.equal(row["h"][r], inf * w1[e, d - 1].sign())
    others = torch.arange(B) != r
    for n in ("h", "y", "dxd"):
        assert torch.equal(row[n][others], clean[n][others]), n
    # a weight of W2: its column of the expert's Y, with the activations' signs
    s = slice(sum(rows[:e]), sum(rows[:e + 1]))
    assert torch.equal(weight["y"][s, 3], inf * clean["h"][s, f - 1].sign())
    mask = torch.ones(B, d, dtype=torch.bool)
    mask[s, 3] = False
    assert torch.equal(weight["y"][mask], clean["y"][mask])
    same = [i for i in range(E) if i != e]
    for n in ("dw1", "dw2"):
        assert torch.equal(weight[n][same], clean[n][same]), n


def test_largest_floats():
    """Products of the largest and of small floats stay what they are."""
    import paper_2508_13337_amd as m
    rows, d, f = [40, 90], 48, 33
    x, w, dy = random_ffn(rows, d, f, torch.float32)
    x = x.sign() * 3.4e38
    w[0], w[1] = w[0] * 1e-32, w[1] * 1e-32
    o = ffn(m, rows, x, w, dy)
    for e, s in enumerate((slice(0, 40), slice(40, 130))):
        for name, a in (("g", w[0]), ("u", w[1])):
            want = x[s].double() @ a[e].double()
            err = (o[name][s].double() - want).abs() / want.pow(2).mean(1, keepdim=True).sqrt()
            assert float(err.max()) < 2.0 ** -16, (name, float(err.max()))


def product(m, x, w):
    """x @ w for float32 [B, K] and [K, N]: the first product of the two-matrix expert with no activation."""
    (B, K), N = x.shape, w.shape[1]
    h, y = torch.empty((B, N), device="cuda"), torch.empty((B, K), device="cuda")
    ws = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_MLP2_FWD, B, K, 1, 1, N, m.XMOE_F32))
    off = torch.tensor([0, B], dtype=torch.int32, device="cuda")
    m.xmoe_expert_mlp2_fwd(x.cuda(), off, w[None].contiguous().cuda(), torch.zeros((1, N, K), device="cuda"), "identity", h, y, ws)
    return h.cpu()


@pytest.mark.parametrize("K", [1, 2, 3, 4, 7, 8, 9, 15, 16, 17, 33, 100])
@pytest.mark.parametrize("B", [70, 3000])
def test_float32_products_round_no_more_than_float32(B, K):
    """A chain of float32 additions rounds each of its K sums by at most 2^-24 of the sum of the terms' magnitudes.  Operands
    of all bits, and ones whose last 16 bits are as large as they can be."""
    import paper_2508_13337_amd as m
    g = torch.Generator().manual_seed(B + K)
    last16 = lambda *s: 1 + 2.0 ** -7 - torch.randint(1, 300, s, generator=g).float() * 2.0 ** -23
    for new in (lambda *s: torch.randn(s, generator=g), last16):
        x, w = new(B, K), new(K, 96)
        err = (product(m, x, w).double() - x.double() @ w.double()).abs()
        assert float((err / (x.double().abs() @ w.double().abs())).max()) <= K * 2.0 ** -24


@pytest.mark.parametrize("K", [7, 40])
@pytest.mark.parametrize("ex,ew", [(-120, 100), (-126, 110), (-140, 120), (-100, -20), (-110, -33), (103, 20), (104, -20), (126, -60),
                                   (40, 39), (41, 40), (60, 60)])
def test_float32_products_of_small_and_large_operands(ex, ew, K):
    """The whole range of float32, subnormal operands and results included: rounded as any other product (as above; a result
    below 2^-126 by half of 2^-149 once more)."""
    import paper_2508_13337_amd as m
    g = torch.Generator().manual_seed(K)
    x, w = ((torch.rand(s, generator=g) + 0.5) * torch.randint(0, 2, s, generator=g).mul(2).sub(1) for s in ((300, K), (K, 96)))
    x, w = (torch.ldexp(t.double(), torch.tensor(e)).float() for t, e in ((x, ex), (w, ew)))
    want = x.double() @ w.double()
    bound = K * 2.0 ** -24 * (x.double().abs() @ w.double().abs()) + (K + 1) * 2.0 ** -150
    assert bool(((product(m, x, w).double() - want).abs() <= bound).all())


# one expert with one, two and three windows of 8192 rows, ties across them; capacities at the windows' edges
@pytest.mark.parametrize("T,cap", [(8192, 8191), (8193, 8192), (16385, 8193), (16385, 16384), (20000, 3), (20000, 12000)])
def test_token_dropping_of_long_segments(T, cap):
    rng = np.random.default_rng(T + cap)
    idx = np.zeros((T, 1), np.int32)
    idx[5::1000] = 1
    for w in (rng.integers(1, 9, (T, 1)).astype(np.float32) / 8, rng.random((T, 1), np.float32)):
        check_capped_eri(run_build_eri(idx, w, 2, max_token_count=cap), oracle.build_eri_capped(idx, w, 2, cap), 2)


@pytest.mark.parametrize("E,k", [(1, 1), (8, 2), (64, 6), (65, 8), (256, 8), (512, 1), (512, 8)])
def test_route_bwd_rows_is_both_passes(E, k):
    import paper_2508_13337_amd as m
    T = 133
    g = torch.Generator().manual_seed(E + k)
    logits, rg = torch.randn(T, E, generator=g).cuda(), torch.randn(T * k, generator=g).cuda()
    idx = i32(torch.rand(T, E, generator=g).topk(k).indices.numpy())
    ros = torch.randperm(T * k, generator=g).int()
    ros[::7] = -1                                        # dropped entries
    ros = ros.cuda()
    new = lambda n: torch.full((T, n), 7.0, device="cuda")
    dw, dl, dw2, dl2 = new(k), new(E), new(k), new(E)
    m.xmoe_combine_bwd_weights(rg, ros, dw)
    m.xmoe_route_bwd(logits, idx, dw, dl)
    m.xmoe_route_bwd_rows(logits, idx, rg, ros, dw2, dl2)
    assert torch.equal(dw, dw2) and torch.equal(dl, dl2)


@pytest.mark.parametrize("E,k", [(8, 8), (40, 7), (64, 64), (65, 8), (200, 8), (512, 64)])
def test_route_selects_every_expert_once(E, k):
    """NaNs of all bit patterns, -1 (all ones) among them, take their place in the order of the bits, as infinities do."""
    import paper_2508_13337_amd as m
    rng = np.random.default_rng(E + k)
    odd = np.array([0xffffffff, 0xfffffffe, 0x7fffffff, 0x7fc00000, 0xffc00000, 0xff800000, 0x7f800000, 0x80000000, 0], np.uint32)
    bits = rng.standard_normal((67, E)).astype(np.float32).view(np.uint32)
    bits[0:40] = rng.choice(odd, (40, E))
    bits[40:44] = 0xffffffff
    bits[44:48, 1:] = 0xffffffff
    bits[48:52, :E - 1] = 0xffffffff
    b = np.where(bits == 0x80000000, np.uint32(0), bits)          # the zeros are one number
    key = np.where(b >> 31, ~b, b | np.uint32(0x80000000)).astype(np.int64)
    want = np.argsort(-key, axis=1, kind="stable")[:, :k]
    logits = torch.from_numpy(bits.view(np.float32)).cuda()
    idx = torch.full((67, k), -1, dtype=torch.int32, device="cuda")
    m.xmoe_route(logits, k, idx, torch.empty((67, k), device="cuda"))
    assert np.array_equal(idx.cpu().numpy(), want)


@pytest.mark.parametrize("E", [64, 65, 127, 129, 256, 257, 512])
def test_tile_maps_of_many_experts(E):
    """Segments of no row up to three tiles, in the forward's and the backward's maps."""
    import paper_2508_13337_amd as m
    rows, d, f = [(e * 37) % 5 if e % 9 else (e * 31) % 150 for e in range(E)], 24, 16
    x, w, dy = random_ffn(rows, d, f, torch.float32)
    o = ffn(m, rows, x, w, dy)
    at = 0
    for e, n in enumerate(rows):
        X, D, W = x[at:at + n].double(), dy[at:at + n].double(), [a[e].double() for a in w]
        G, U = X @ W[0], X @ W[1]
        S = torch.sigmoid(G)
        A, dA = G * S * U, D @ W[2].t()
        dG, dU = dA * U * S * (1 + G * (1 - S)), dA * G * S
        for name, got, want in (("y", o["y"][at:at + n], A @ W[2]), ("dxd", o["dxd"][at:at + n], dG @ W[0].t() + dU @ W[1].t()),
                                ("dwg", o["dwg"][e], X.t() @ dG), ("dwu", o["dwu"][e], X.t() @ dU), ("dwd", o["dwd"][e], A.t() @ D)):
            if want.numel():
                err = (got.double() - want).abs().max() / want.abs().max().clamp_min(1e-30) if want.any() else got.abs().max()
                assert float(err) < 2.0 ** -16, (name, e, n, float(err))
        at += n
