"""The general matrix-core tiles (float32, and bf16 widths that are no multiple of 8 or operands that are not 16-byte aligned;
bf16 rows start two bytes behind such an address here) at the sizes where they can go
wrong: K of less than one step, one past a step and one element past a 16-byte vector; columns that end inside a
four-column load or are fewer than four; row segments on both sides of every 32-row block and of both tile heights;
leading dimensions of every residue, so that loads start unaligned.  Expert MLP forward and backward with gathered
rows, against the oracle in float64."""
import numpy as np
import pytest
import torch

import oracle
import xmoe_inputs as xi
from gpu_util import launched, to_dev, to_host, torch_dtype

pytestmark = pytest.mark.gpu

SHORT = (1, 0, 31, 32, 33, 63, 64, 65, 127, 128, 129)
# experts with more than 96 rows on average and enough of them for the 128 x 128 tile of the row products
LONG = (2100, 0, 1, 2049, 4000)
# one more of them: the weight gradients take 128 x 128 tiles too (3 matrices x 6 experts x 30 tiles >= 512; the two-matrix
# expert's, 2 x 9 x 30)
LONG6 = LONG + (130,)
LONG9 = LONG6 + (0, 95, 700)


def guarded(shape, dtype):
    """A tensor with 256 marked elements before and behind it: (tensor, check that the marks stand)."""
    n = int(np.prod(shape))
    buf = torch.full((n + 512,), 3.0, dtype=dtype, device="cuda")

    def check():
        assert bool((buf[:256] == 3.0).all()) and bool((buf[256 + n:] == 3.0).all())

    return buf[256:256 + n].view(shape), check


def to_dev_unaligned(a, dtype):
    t = to_dev(a, dtype)
    if dtype == "f32":
        return t
    u = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape)
    return u.copy_(t)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,f,rows", [(1, 1, SHORT), (3, 5, SHORT), (7, 2, SHORT), (31, 33, SHORT), (66, 127, SHORT),
                                      (130, 61, SHORT), (129, 200, SHORT), (72, 8, SHORT), (517, 645, LONG),
                                      (520, 648, LONG), (517, 645, LONG6), (520, 648, LONG6)])
def test_expert_ffn_any_width(d, f, rows, dtype):
    import paper_2508_13337_amd as m
    rng = np.random.default_rng(1000 * d + f)
    T, E = 400, len(rows)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    B = int(off[-1])
    tdt = torch_dtype(dtype)

    def draw(shape, scale=1.0):
        return xi.round_to_storage((rng.standard_normal(shape) * scale).astype(np.float32), dtype)

    x, dout = draw((T, d)), draw((T, d))
    tok = rng.integers(0, T, size=B).astype(np.int32)
    cw = rng.random(B).astype(np.float32)
    wg, wu, wd = draw((E, d, f), d ** -0.5), draw((E, d, f), d ** -0.5), draw((E, f, d), f ** -0.5)
    ti, to = torch.from_numpy(tok).cuda(), torch.from_numpy(off).cuda()
    code = m.dtype_code(tdt)
    ws = m.alloc_workspace(max(m.xmoe_workspace_bytes(m.WS_FFN_FWD, B, d, E, 1, f, code),
                               m.xmoe_workspace_bytes(m.WS_FFN_BWD, B, d, E, 1, f, code)))
    out = {n: guarded(s, tdt) for n, s in dict(g=(B, f), u=(B, f), y=(B, d), dxd=(B, d), dwg=(E, d, f), dwu=(E, d, f),
                                               dwd=(E, f, d)).items()}
    row_grad, row_ok = guarded((B,), torch.float32)
    t = {n: v[0] for n, v in out.items()}
    xt, dt_, wgt, wut, wdt = to_dev_unaligned(x, dtype), *(to_dev(a, dtype) for a in (dout, wg, wu, wd))
    m.xmoe_prof_reset()
    m.xmoe_prof_enable(True)
    m.xmoe_expert_ffn_fwd(xt, to, wgt, wut, wdt, t["g"], t["u"], t["y"], ws, row_index=ti)
    m.xmoe_expert_ffn_bwd(xt, t["g"], t["u"], dt_, to, wgt, wut, wdt, t["dxd"], t["dwg"], t["dwu"], t["dwd"], ws,
                          row_index=ti, dy_row_index=ti, dy_row_scale=torch.from_numpy(cw).cuda(),
                          dy_row_scale_grad=row_grad)
    torch.cuda.synchronize()
    launched = set(m.xmoe_prof_read())
    m.xmoe_prof_enable(False)
    m.xmoe_prof_reset()
    assert {"ffn_gateup_mfma_kernel", "ffn_down_mfma_kernel", "ffn_dact_mfma_kernel", "ffn_dx_mfma_kernel",
            "ffn_wgrad_mfma_kernel"} <= launched, launched
    for _, check in out.values():
        check()
    row_ok()
    # Bounds: every stored value rounds by at most u of itself, every float32 sum of n products by at most n * 2^-24 of
    # the sum of their magnitudes (h covers the few roundings of the activation), and a factor's error goes into a
    # product with the other factor's magnitude.  Narrow rows cancel, so nothing is taken relative to a row's norm.
    u = 2.0 ** -24 if dtype == "f32" else 2.0 ** -8
    eps, h = 2.0 ** -24, 16
    w64 = [a.astype(np.float64) for a in (wg, wu, wd)]
    Xd, dY0, sc = x.astype(np.float64)[tok], dout.astype(np.float64)[tok], cw.astype(np.float64)[:, None]
    Y, G, U = oracle.expert_ffn_fwd(Xd, off, *w64)
    Gs, Us = to_host(t["g"]), to_host(t["u"])          # the stored activations the backward starts from
    dxd, dwg, dwu, dwd = oracle.expert_ffn_bwd(Xd, Gs, Us, sc * dY0, off, *w64)

    def within(name, got, want, bound):
        over = np.abs(got - want) - (bound * 1.01 + u * np.abs(want) + 1e-30)
        assert (over <= 0).all(), (name, float(over.max()), np.argwhere(over > 0)[:4].tolist())

    rg = row_grad.cpu().numpy().astype(np.float64)
    got = {n: to_host(v) for n, v in t.items()}
    for e in range(E):
        s = slice(off[e], off[e + 1])
        n = rows[e]
        if n == 0:
            assert not t["dwg"][e].any() and not t["dwu"][e].any() and not t["dwd"][e].any()
            continue
        X, D, c = np.abs(Xd[s]), np.abs(dY0[s]), sc[s]
        Wg, Wu, Wd = (np.abs(w[e]) for w in w64)
        eG, eU = (d + h) * eps * (X @ Wg), (d + h) * eps * (X @ Wu)
        within("g", got["g"][s], G[s], eG)
        within("u", got["u"][s], U[s], eU)
        silu = G[s] / (1 + np.exp(-G[s]))
        A, eA = np.abs(silu * U[s]), 1.1 * eG * np.abs(U[s]) + np.abs(silu) * eU     # |silu'| < 1.1
        eA = eA + (u + h * eps) * A
        within("y", got["y"][s], Y[s], eA @ Wd + (f + h) * eps * (A @ Wd))
        sg = 1 / (1 + np.exp(-Gs[s]))
        S = Gs[s] * sg
        kg, ku, ka = np.abs(Us[s] * sg * (1 + Gs[s] * (1 - sg))), np.abs(S), np.abs(S * Us[s])
        dA0 = dY0[s] @ w64[2][e].T
        e0 = (d + h) * eps * (D @ Wd.T)
        dG, dU, eS = c * np.abs(dA0) * kg, c * np.abs(dA0) * ku, (u + h * eps) * c * ka
        edG, edU = c * e0 * kg + (u + h * eps) * dG, c * e0 * ku + (u + h * eps) * dU
        within("dxd", got["dxd"][s], dxd[s], edG @ Wg.T + edU @ Wu.T + (2 * f + h) * eps * (dG @ Wg.T + dU @ Wu.T))
        within("dwg", got["dwg"][e], dwg[e], X.T @ edG + (n + h) * eps * (X.T @ dG))
        within("dwu", got["dwu"][e], dwu[e], X.T @ edU + (n + h) * eps * (X.T @ dU))
        within("dwd", got["dwd"][e], dwd[e], eS.T @ D + (n + h) * eps * ((c * ka).T @ D))
        within("row_grad", rg[s], (dA0 * S * Us[s]).sum(1), (e0 * ka).sum(1) + (f + h) * eps * (np.abs(dA0) * ka).sum(1))


@pytest.mark.parametrize("dtype,act", [("f32", "gelu"), ("f32", "silu"), ("bf16", "gelu"), ("bf16", "identity")])
@pytest.mark.parametrize("d,f,rows", [(3, 5, SHORT), (66, 127, SHORT), (130, 61, SHORT), (517, 645, LONG9)])
def test_expert_mlp2_any_width(d, f, rows, dtype, act):
    """The two-matrix expert on the same tiles; bounds as above, with |act'| <= 1.13 and |act''| <= 1."""
    import paper_2508_13337_amd as m
    rng = np.random.default_rng(2000 * d + f)
    T, E = 400, len(rows)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    B = int(off[-1])
    tdt = torch_dtype(dtype)

    def draw(shape, scale=1.0):
        return xi.round_to_storage((rng.standard_normal(shape) * scale).astype(np.float32), dtype)

    x, dout = draw((T, d)), draw((T, d))
    tok = rng.integers(0, T, size=B).astype(np.int32)
    cw = rng.random(B).astype(np.float32)
    w1, w2 = draw((E, d, f), d ** -0.5), draw((E, f, d), f ** -0.5)
    ti, to = torch.from_numpy(tok).cuda(), torch.from_numpy(off).cuda()
    code = m.dtype_code(tdt)
    ws = m.alloc_workspace(max(m.xmoe_workspace_bytes(m.WS_MLP2_FWD, B, d, E, 1, f, code),
                               m.xmoe_workspace_bytes(m.WS_MLP2_BWD, B, d, E, 1, f, code)))
    out = {n: guarded(s, tdt) for n, s in dict(h=(B, f), y=(B, d), dxd=(B, d), dw1=(E, d, f), dw2=(E, f, d)).items()}
    row_grad, row_ok = guarded((B,), torch.float32)
    t = {n: v[0] for n, v in out.items()}
    xt, dt_, w1t, w2t = to_dev_unaligned(x, dtype), *(to_dev(a, dtype) for a in (dout, w1, w2))

    def call():
        m.xmoe_expert_mlp2_fwd(xt, to, w1t, w2t, act, t["h"], t["y"], ws, row_index=ti)
        m.xmoe_expert_mlp2_bwd(xt, t["h"], dt_, to, w1t, w2t, act, t["dxd"], t["dw1"], t["dw2"], ws, row_index=ti,
                               dy_row_index=ti, dy_row_scale=torch.from_numpy(cw).cuda(), dy_row_scale_grad=row_grad)

    kernels = launched(m, call)
    assert {"mlp2_up_mfma_kernel", "mlp2_dact_mfma_kernel", "ffn_wgrad_mfma_kernel"} <= kernels, kernels
    for _, check in out.values():
        check()
    row_ok()
    u = 2.0 ** -24 if dtype == "f32" else 2.0 ** -8
    eps, h = 2.0 ** -24, 16
    w64 = [a.astype(np.float64) for a in (w1, w2)]
    Xd, dY0, sc = x.astype(np.float64)[tok], dout.astype(np.float64)[tok], cw.astype(np.float64)[:, None]
    Y, H = oracle.expert_mlp2_fwd(Xd, off, *w64, act)
    Hs = to_host(t["h"])                               # the stored activations the backward starts from
    dxd, dw1, dw2 = oracle.expert_mlp2_bwd(Xd, Hs, sc * dY0, off, *w64, act)

    def within(name, got, want, bound):
        over = np.abs(got - want) - (bound * 1.01 + u * np.abs(want) + 1e-30)
        assert (over <= 0).all(), (name, float(over.max()), np.argwhere(over > 0)[:4].tolist())

    rg = row_grad.cpu().numpy().astype(np.float64)
    got = {n: to_host(v) for n, v in t.items()}
    for e in range(E):
        s = slice(off[e], off[e + 1])
        n = rows[e]
        if n == 0:
            assert not t["dw1"][e].any() and not t["dw2"][e].any()
            continue
        X, D, c = np.abs(Xd[s]), np.abs(dY0[s]), sc[s]
        W1, W2 = (np.abs(w[e]) for w in w64)
        eH = (d + h) * eps * (X @ W1)
        within("h", got["h"][s], H[s], eH)
        act64, act_h = oracle.activation(act, H[s]), oracle.activation(act, Hs[s])
        # the activation itself: a few roundings of H-sized numbers (gelu and silu are H times a factor below 1)
        A, eA = np.abs(act64), 1.13 * eH + h * eps * np.abs(H[s])
        eA = eA + u * A
        within("y", got["y"][s], Y[s], eA @ W2 + (f + h) * eps * (A @ W2))
        kg, ka = np.abs(oracle.activation_grad(act, Hs[s])), np.abs(act_h)
        sa = h * eps * np.abs(Hs[s])
        dA0 = dY0[s] @ w64[1][e].T
        e0 = (d + h) * eps * (D @ W2.T)
        dH, eS = c * np.abs(dA0) * kg, c * (u * ka + sa)
        edH = c * e0 * kg + u * dH + h * eps * c * np.abs(dA0) * 1.13
        within("dxd", got["dxd"][s], dxd[s], edH @ W1.T + (f + h) * eps * (dH @ W1.T))
        within("dw1", got["dw1"][e], dw1[e], X.T @ edH + (n + h) * eps * (X.T @ dH))
        within("dw2", got["dw2"][e], dw2[e], eS.T @ D + (n + h) * eps * ((c * ka).T @ D))
        within("row_grad", rg[s], (dA0 * act_h).sum(1),
               (e0 * ka + np.abs(dA0) * sa).sum(1) + (f + h) * eps * (np.abs(dA0) * ka).sum(1))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_rows_bits_do_not_depend_on_the_row_count(dtype):
    """The same tokens in a call that takes the small tiles and among enough others for the large ones."""
    import paper_2508_13337_amd as m
    T, d, f, few, many = 400, 300, 200, (1, 33, 0, 64), (4000, 4300, 90, 8500)
    g = torch.Generator().manual_seed(7)
    tdt = torch_dtype(dtype)
    x, wg, wu, wd = (torch.randn(s, generator=g).to(tdt).cuda() * 0.1
                     for s in ((T, d), (4, d, f), (4, d, f), (4, f, d)))
    more = [torch.randint(0, T, (n,), generator=g, dtype=torch.int32) for n in many]
    runs = []
    for rows, index in ((few, [i[:n] for i, n in zip(more, few)]), (many, more)):
        off = torch.tensor([0] + list(torch.tensor(rows).cumsum(0)), dtype=torch.int32).cuda()
        B = sum(rows)
        out = [torch.empty((B, n), dtype=tdt, device="cuda") for n in (f, f, d)]
        ws = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_FFN_FWD, B, d, 4, 1, f, m.dtype_code(tdt)))
        m.xmoe_expert_ffn_fwd(x, off, wg, wu, wd, *out, ws, row_index=torch.cat(index).cuda())
        runs.append((off.tolist(), [o.cpu() for o in out]))
    (o1, a), (o2, b) = runs
    for p, q in zip(a, b):
        for e, n in enumerate(few):
            assert torch.equal(p[o1[e]:o1[e] + n], q[o2[e]:o2[e] + n]), e
