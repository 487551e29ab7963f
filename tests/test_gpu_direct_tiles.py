"""The 128 x 128 tiles with direct-to-LDS loads (xmoe_ffn_direct.hip): segments at the edges of their row blocks, K of
less than one 64-wide unit and with ragged ends, output tiles of every 8-column remainder, both sides of the rules that
choose them, and the bits of the 256-row kernels.

Tolerance: every stored result is one float32-accumulated product of bf16 operands, rounded once (2^-9 relative).  The
reference rounds the stored factors (A, dG, dU) as the kernels do, so that an odd rounding of a factor is all they differ
by.  Results are held to 2^-6 of the row's (weight gradients: the matrix's) root mean square
or of the value itself; the row scales' gradient is a float32 sum."""
import pytest
import torch

from gpu_util import launched

pytestmark = pytest.mark.gpu

ROWS = [1, 0, 31, 32, 33, 63, 64, 65, 127, 128, 129, 200, 7]


def inputs(rows, d, f, matrices):
    g = torch.Generator().manual_seed(sum(rows) + d + 3 * f + matrices)
    E, B, T = len(rows), sum(rows), 61
    off = torch.tensor([0] + list(torch.tensor(rows).cumsum(0)), dtype=torch.int32)
    x, dout = (torch.randn((T, d), generator=g).bfloat16() for _ in range(2))
    idx = torch.randint(0, T, (B,), generator=g, dtype=torch.int32)
    scale = torch.rand(B, generator=g)
    w = [(torch.randn((E, f, d) if i == matrices - 1 else (E, d, f), generator=g) * (f if i == matrices - 1 else d) ** -0.5)
         .bfloat16() for i in range(matrices)]
    return off, x, dout, idx, scale, w


def run(m, rows, d, f, expert, gathered=True, scaled=True):
    """Forward and backward: {name: tensor} on the host, and the kernels launched by either."""
    off, x, dout, idx, scale, w = inputs(rows, d, f, 3 if expert == "swiglu" else 2)
    B, E = sum(rows), len(rows)
    X, D = (t if gathered else t[idx.long()] for t in (x, dout))
    new = lambda *s: torch.full(s, 7.0, dtype=torch.bfloat16, device="cuda")
    t = {"y": new(B + 1, d), "dxd": new(B + 1, d)}
    t.update({n: new(B + 1, f) for n in (("g", "u") if expert == "swiglu" else ("h",))})
    t.update({"dw%d" % i: new(*a.shape) for i, a in enumerate(w)})
    t["rg"] = torch.full((B + 1,), 7.0, device="cuda")
    o = {n: a[:B] if a.shape[0] == B + 1 else a for n, a in t.items()}
    two = expert != "swiglu"
    ws = m.alloc_workspace(max(m.xmoe_workspace_bytes(op, B, d, E, 1, f, m.XMOE_BF16)
                               for op in ((m.WS_MLP2_FWD, m.WS_MLP2_BWD) if two else (m.WS_FFN_FWD, m.WS_FFN_BWD))))
    xc, dc, oc, wc, ic = X.cuda(), D.cuda(), off.cuda(), [a.cuda() for a in w], idx.cuda() if gathered else None
    kw = dict(row_index=ic, dy_row_index=ic, dy_row_scale=scale.cuda() if gathered and scaled else None,
              dy_row_scale_grad=o["rg"])
    if two:
        k1 = launched(m, lambda: m.xmoe_expert_mlp2_fwd(xc, oc, *wc, expert, o["h"], o["y"], ws, row_index=ic))
        k2 = launched(m, lambda: m.xmoe_expert_mlp2_bwd(xc, o["h"], dc, oc, *wc, expert, o["dxd"], o["dw0"], o["dw1"], ws,
                                                        **kw))
    else:
        k1 = launched(m, lambda: m.xmoe_expert_ffn_fwd(xc, oc, *wc, o["g"], o["u"], o["y"], ws, row_index=ic))
        k2 = launched(m, lambda: m.xmoe_expert_ffn_bwd(xc, o["g"], o["u"], dc, oc, *wc, o["dxd"], o["dw0"], o["dw1"],
                                                       o["dw2"], ws, **kw))
    host = {n: a.cpu() for n, a in t.items()}
    assert all(bool((a[B] == 7.0).all()) for n, a in host.items() if a.shape[0] == B + 1)   # nothing behind the last row
    return {n: a[:B] if a.shape[0] == B + 1 else a for n, a in host.items()}, k1, k2


def close(name, got, want, dims=-1, tol=2.0 ** -6):
    rms = want.pow(2).mean(dim=dims, keepdim=True).sqrt()
    err = ((got.double() - want).abs() / torch.maximum(want.abs(), rms).clamp_min(1e-30)).max()
    assert float(err) <= tol, (name, float(err))


def act64(name, h):
    if name == "identity":
        return h, torch.ones_like(h)
    if name == "gelu":
        cdf = 0.5 * torch.erfc(-h / 2 ** 0.5)
        return h * cdf, cdf + h * torch.exp(-0.5 * h * h) / (2 * torch.pi) ** 0.5
    s = torch.sigmoid(h)
    return h * s, s * (1 + h * (1 - s))


def check(rows, d, f, expert, o, gathered=True, scaled=True):
    off, x, dout, idx, scale, w = inputs(rows, d, f, 3 if expert == "swiglu" else 2)
    c = scale.double() if gathered and scaled else torch.ones(sum(rows), dtype=torch.float64)
    for e, n in enumerate(rows):
        s = slice(int(off[e]), int(off[e + 1]))
        if n == 0:
            assert not any(bool(o["dw%d" % i][e].any()) for i in range(len(w)))
            continue
        X, D, cs = x[idx[s].long()].double(), dout[idx[s].long()].double(), c[s][:, None]
        W = [a[e].double() for a in w]
        if expert == "swiglu":
            close("g", o["g"][s], X @ W[0])
            close("u", o["u"][s], X @ W[1])
            G, U = o["g"][s].double(), o["u"][s].double()     # the backward starts from the stored activations
            S, dS = act64("silu", G)
            A, back = S * U, lambda dA: [dA * U * dS, dA * S]
            S1, _ = act64("silu", X @ W[0])
            A1 = S1 * (X @ W[1])
        else:
            close("h", o["h"][s], X @ W[0])
            A, dS = act64(expert, o["h"][s].double())
            A1, back = act64(expert, X @ W[0])[0], lambda dA: [dA * dS]
        close("y", o["y"][s], A1.bfloat16().double() @ W[-1])
        P = D @ W[-1].t()
        close("rg", o["rg"][s], (P * A).sum(1), dims=0, tol=1e-4)
        g = [v.bfloat16().double() for v in back(cs * P)]
        close("dxd", o["dxd"][s], sum(v @ a.t() for v, a in zip(g, W)))
        close("dw last", o["dw%d" % (len(w) - 1)][e], (cs * A).bfloat16().double().t() @ D, dims=(0, 1))
        for i, v in enumerate(g):
            close("dw%d" % i, o["dw%d" % i][e], X.t() @ v, dims=(0, 1))


@pytest.mark.parametrize("expert,gathered,scaled", [("swiglu", True, True), ("swiglu", False, False), ("swiglu", True, False),
                                                    ("gelu", True, True), ("silu", False, False), ("identity", True, True)])
@pytest.mark.parametrize("d,f", [(256, 256), (448, 320)])
def test_multiples_of_64(d, f, expert, gathered, scaled):
    import paper_2508_13337_amd as m
    o, k1, k2 = run(m, ROWS, d, f, expert, gathered, scaled)
    up = "ffn_gateup" if expert == "swiglu" else "mlp2_up"
    da = "ffn_dact" if expert == "swiglu" else "mlp2_dact"
    assert k1 == {"tile_map_kernel", up + "_direct_kernel", "ffn_down_direct_kernel"}, k1
    assert {da + "_direct_kernel", "ffn_dx_direct_kernel", "ffn_wgrad_direct_kernel"} <= k2, k2
    check(ROWS, d, f, expert, o, gathered, scaled)


# K of less than a unit, ending inside its first and second half and inside a K-strided tile; one, two and more output tiles
@pytest.mark.parametrize("expert", ["swiglu", "gelu"])
@pytest.mark.parametrize("d,f", [(8, 8), (8, 136), (72, 40), (104, 328), (264, 120), (328, 200)])
@pytest.mark.parametrize("rows", [[1, 0, 30, 1, 3, 2], ROWS, [300, 0, 1000, 129] + [96] * 12, [6200, 0, 6000, 129]],
                         ids=["scarce", "few", "many", "large"])
def test_multiples_of_8(rows, d, f, expert):
    import paper_2508_13337_amd as m
    o, k1, k2 = run(m, rows, d, f, expert)
    up, da = ("ffn_gateup", "ffn_dact") if expert == "swiglu" else ("mlp2_up", "mlp2_dact")
    assert k1 == {"tile_map_kernel", up + "_direct_kernel", "ffn_down_direct_kernel"}, k1
    B, E = sum(rows), len(rows)
    blocks = E * -(-(-(-B // E)) // 64) * -(-max(d, f) // 64)
    rows_by = "direct" if B >= 24 * E and blocks > 512 else "mfma"
    assert {da + "_%s_kernel" % rows_by, "ffn_dx_%s_kernel" % rows_by,
            "ffn_wgrad_%s_kernel" % ("direct" if B >= 12 * E else "mfma")} <= k2, k2
    check(rows, d, f, expert, o)


@pytest.mark.parametrize("expert", ["swiglu", "identity"])
@pytest.mark.parametrize("rows", [[1200, 0, 1001, 63] * 12 + [3000] * 16, [2700, 1, 0, 2300]], ids=["many", "few"])
def test_long_segments(rows, expert):
    """Weight gradients of widths that are no multiple of 64: long segments, with many tiles and with few."""
    import paper_2508_13337_amd as m
    d, f = (264, 392) if expert == "swiglu" else (520, 392)
    o, _, k2 = run(m, rows, d, f, expert)
    assert {"ffn_wgrad_direct_kernel", "ffn_dx_direct_kernel"} <= k2 and not any("dma" in k for k in k2), k2
    check(rows, d, f, expert, o)


def test_bits_of_the_256_row_kernels():
    """The same rows in a call of few tiles and among so many that the 256-row kernels take it."""
    import paper_2508_13337_amd as m
    d, f, few, many = 320, 256, [70, 1, 0, 129], [6000, 5000, 4097, 8000]
    g = torch.Generator().manual_seed(3)
    x = torch.randn((61, d), generator=g).bfloat16().cuda()
    w = [(torch.randn(s, generator=g) * 0.06).bfloat16().cuda() for s in ((64, d, f), (64, d, f), (64, f, d))]
    long = [torch.randint(0, 61, (n,), generator=g, dtype=torch.int32) for n in many]
    outs = []
    for rows in (few, many):
        rows64 = rows + [0 if rows is few else 4500] * 60
        idx = torch.cat([i[:n] for i, n in zip(long, rows)] + [torch.zeros(sum(rows64[4:]), dtype=torch.int32)])
        off = torch.tensor([0] + list(torch.tensor(rows64).cumsum(0)), dtype=torch.int32)
        # few rows on average would take the few-row kernels: the first four experts alone
        E = 4 if rows is few else 64
        B = int(off[E])
        o = [torch.empty((B, n), dtype=torch.bfloat16, device="cuda") for n in (f, f, d)]
        ws = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_FFN_FWD, B, d, E, 1, f, m.XMOE_BF16))
        k = launched(m, lambda: m.xmoe_expert_ffn_fwd(x, off[:E + 1].cuda(), *(a[:E] for a in w), *o, ws,
                                                      row_index=idx[:B].cuda()))
        outs.append((off.tolist(), [t.cpu() for t in o], k))
    assert "ffn_gateup_direct_kernel" in outs[0][2] and "ffn_gateup_dma_kernel" in outs[1][2], (outs[0][2], outs[1][2])
    for p, q in zip(outs[0][1], outs[1][1]):
        for e, n in enumerate(few):
            assert torch.equal(p[outs[0][0][e]:][:n], q[outs[1][0][e]:][:n]), e


@pytest.mark.parametrize("expert", ["swiglu", "gelu"])
@pytest.mark.parametrize("d,f,E", [(320, 256, 64), (328, 200, 4)])
def test_backward_bits_of_the_other_kernels(d, f, E, expert):
    """A row's gradient, and that of its scale, from both sides of the rules: widths of 64, few tiles of 128 rows and many of
    256; widths of 8, the register-staged tiles and these."""
    import paper_2508_13337_amd as m
    few, many = [70, 1, 0, 129], [6000, 5000, 4097, 8000]
    g = torch.Generator().manual_seed(d)
    r = lambda *s: torch.randn(s, generator=g).bfloat16()
    n_mat = 3 if expert == "swiglu" else 2
    w = [(r(E, f, d) if i == n_mat - 1 else r(E, d, f)) * 0.06 for i in range(n_mat)]
    w = [a.cuda() for a in w]
    x, dy = r(61, d).cuda(), r(61, d).cuda()
    idx = [torch.randint(0, 61, (n,), generator=g, dtype=torch.int32) for n in many]
    scale, acts = [torch.rand(n, generator=g) for n in many], [[r(n, f) for n in many] for _ in range(n_mat - 1)]
    outs = []
    for rows in (few, many):
        n_e = E if rows is many else 4
        rest = [4500] * (n_e - 4)
        B = sum(rows) + sum(rest)
        off = torch.tensor([0] + list(torch.tensor(rows + rest).cumsum(0)), dtype=torch.int32)
        rows_of = lambda t: torch.cat([a[:n] for a, n in zip(t, rows)] + [a[:1].expand(sum(rest), *a.shape[1:]) for a in t[:1]])
        ic, sc, *saved = (rows_of(t).cuda() for t in (idx, scale, *acts))
        o = [torch.empty((B, d), dtype=torch.bfloat16, device="cuda")] + [torch.empty_like(a[:n_e]) for a in w]
        rg = torch.empty(B, device="cuda")
        kw = dict(row_index=ic, dy_row_index=ic, dy_row_scale=sc, dy_row_scale_grad=rg)
        op = m.WS_FFN_BWD if expert == "swiglu" else m.WS_MLP2_BWD
        ws = m.alloc_workspace(m.xmoe_workspace_bytes(op, B, d, n_e, 1, f, m.XMOE_BF16))
        wc = [a[:n_e] for a in w]
        if expert == "swiglu":
            k = launched(m, lambda: m.xmoe_expert_ffn_bwd(x, *saved, dy, off.cuda(), *wc, *o, ws, **kw))
        else:
            k = launched(m, lambda: m.xmoe_expert_mlp2_bwd(x, *saved, dy, off.cuda(), *wc, expert, *o, ws, **kw))
        outs.append((off.tolist(), o[0].cpu(), rg.cpu(), k))
    (o1, dx1, rg1, k1), (o2, dx2, rg2, k2) = outs
    direct = "ffn_dact_direct_kernel" if expert == "swiglu" else "mlp2_dact_direct_kernel"
    assert (direct in k1) == (d % 64 == 0) and (direct in k2) != (d % 64 == 0), (k1, k2)
    for e, n in enumerate(few):
        assert torch.equal(dx1[o1[e]:][:n], dx2[o2[e]:][:n]), e
        assert torch.equal(rg1[o1[e]:][:n], rg2[o2[e]:][:n]), e


@pytest.mark.parametrize("expert", ["swiglu", "identity"])
@pytest.mark.parametrize("f", [200, 264])
def test_an_infinite_last_column_is_counted_once(f, expert):
    """An infinite weight of the last valid column makes the gradients of the row scales infinite, not NaN: the columns behind
    it, which repeat it, take no part in them."""
    import paper_2508_13337_amd as m
    rows, d = [3000, 129, 0, 4000], 264
    E, B, g = 4, sum(rows), torch.Generator().manual_seed(f)
    r = lambda *s: torch.randn(s, generator=g).bfloat16()
    off = torch.tensor([0] + list(torch.tensor(rows).cumsum(0)), dtype=torch.int32).cuda()
    n_mat = 3 if expert == "swiglu" else 2
    w = [r(E, f, d) if i == n_mat - 1 else r(E, d, f) for i in range(n_mat)]
    w[-1][:, f - 1, 7] = float("inf")
    dy, acts = r(B, d), [r(B, f) for _ in range(n_mat - 1)]
    o = [torch.empty((B, d), dtype=torch.bfloat16, device="cuda")] + [torch.empty_like(a, device="cuda") for a in w]
    rg, ic = torch.empty(B, device="cuda"), torch.arange(B, dtype=torch.int32, device="cuda")
    ws = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_FFN_BWD if n_mat == 3 else m.WS_MLP2_BWD, B, d, E, 1, f, m.XMOE_BF16))
    kw = dict(row_index=ic, dy_row_index=ic, dy_row_scale_grad=rg)
    args = [a.cuda() for a in acts] + [dy.cuda(), off] + [a.cuda() for a in w]
    if expert == "swiglu":
        k = launched(m, lambda: m.xmoe_expert_ffn_bwd(r(B, d).cuda(), *args, *o, ws, **kw))
    else:
        k = launched(m, lambda: m.xmoe_expert_mlp2_bwd(r(B, d).cuda(), *args, expert, *o, ws, **kw))
    assert ("ffn_dact_direct_kernel" if expert == "swiglu" else "mlp2_dact_direct_kernel") in k, k
    sign = dy[:, 7].float().sign() * torch.stack([a[:, f - 1].float().sign() for a in acts]).prod(0)
    assert torch.equal(rg.cpu(), float("inf") * sign)


@pytest.mark.parametrize("E,d,f,rows,fwd,bwd,wgrads", [
    (4, 256, 256, 129, True, True, True), (4, 192, 256, 129, False, False, False), (4, 256, 192, 129, False, False, False),
    (64, 256, 256, 64 * 800, False, True, True), (64, 256, 256, 64 * 3200, False, False, False),
    (8, 2048, 2048, 8 * 60, True, True, True), (10, 2048, 2560, 600, True, True, False)])
def test_both_sides_of_the_rules(E, d, f, rows, fwd, bwd, wgrads):
    import paper_2508_13337_amd as m
    count = [rows // E + (e < rows % E) for e in range(E)]
    _, k1, k2 = run(m, count, d, f, "swiglu")
    assert ("ffn_gateup_direct_kernel" in k1) == fwd and ("ffn_gateup_dma_kernel" in k1) != fwd, k1
    assert ("ffn_dact_direct_kernel" in k2) == bwd and ("ffn_rowgemm_dma_kernel<true>" in k2) != bwd, k2
    # dX is part of the weight gradients' launch only where no kernel of its own computes it
    assert ("ffn_wgrad_direct_kernel" in k2) == wgrads and ("ffn_dx_direct_kernel" in k2) == bwd, k2
    assert ("ffn_bwd_wgrads_dma_kernel" in k2) == (bwd and not wgrads) and ("ffn_bwd_rest_dma_kernel" in k2) != bwd, k2


@pytest.mark.parametrize("E,d,f,mean,direct", [(32, 2048, 2560, 40, True), (32, 2048, 2560, 73, False), (80, 2048, 1152, 72, True),
                                               (64, 2048, 1792, 40, False), (64, 1536, 1536, 96, True), (64, 1536, 1536, 97, False)])
def test_forward_rule_for_half_empty_tiles(E, d, f, mean, direct):
    """By the size of the weights and the mean row count alone."""
    import paper_2508_13337_amd as m
    B = E * mean
    off = torch.arange(0, B + 1, mean, dtype=torch.int32).cuda()
    new = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    ws = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_FFN_FWD, B, d, E, 1, f, m.XMOE_BF16))
    w = new(E, d, f), new(E, d, f), new(E, f, d)
    k = launched(m, lambda: m.xmoe_expert_ffn_fwd(new(B, d), off, *w, new(B, f), new(B, f), new(B, d), ws))
    assert ("ffn_gateup_direct_kernel" in k) == direct and ("ffn_gateup_dma_kernel" in k) != direct, k


@pytest.mark.parametrize("E,d,f,B,rows,wgrads", [(87, 328, 200, 24 * 87, True, True), (87, 328, 200, 24 * 87 - 1, False, True),
                                                 (85, 328, 200, 64 * 85, False, True), (86, 200, 328, 64 * 86, True, True),
                                                 (9, 2040, 200, 128 * 9, True, True), (8, 2040, 200, 128 * 8, False, True),
                                                 (200, 328, 200, 12 * 200, False, True), (200, 328, 200, 12 * 200 - 1, False, False)])
def test_backward_rules_of_widths_of_8(E, d, f, B, rows, wgrads):
    """Which kernels take the row products (more than 512 staged tiles, 24 rows per expert) and the weight gradients (12)."""
    import paper_2508_13337_amd as m
    off = torch.tensor([min(B, -(-B // E) * e) for e in range(E + 1)], dtype=torch.int32).cuda()
    new = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    ws = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_FFN_BWD, B, d, E, 1, f, m.XMOE_BF16))
    w = new(E, d, f), new(E, d, f), new(E, f, d)
    k = launched(m, lambda: m.xmoe_expert_ffn_bwd(new(B, d), new(B, f), new(B, f), new(B, d), off, *w, new(B, d),
                                                  *(torch.empty_like(a) for a in w), ws))
    for name in ("ffn_dact_%s_kernel", "ffn_dx_%s_kernel"):
        assert (name % "direct" in k) == rows and (name % "mfma" in k) != rows, k
    assert ("ffn_wgrad_direct_kernel" in k) == wgrads and ("ffn_wgrad_mfma_kernel" in k) != wgrads, k
