"""Forward products of experts with few rows (at most 64 on average): segments at the edges of a 32- and a 64-row block,
widths that fill a 128-column tile and widths that do not, K that splits unevenly over a block's four waves.

Tolerance: G, U, H and the activations are one float32-accumulated product rounded to bf16 (2^-9 relative) against a
float64 product of the same operands; an element that cancels to below the RMS is held to that share of the RMS."""
import pytest
import torch

pytestmark = pytest.mark.gpu

ROWS = {
    "edges": [0, 1, 31, 32, 33, 63, 64, 65, 0],
    "one long": [1, 0, 200, 0, 3, 0],      # 204 rows, 34 on average: four row tiles of one expert
    "single": [1],
}
WIDTHS = [(64, 64), (128, 192), (320, 64), (192, 448), (1024, 704)]   # d, f


def close(got, want, tol=2.0 ** -7):
    err = (got.double() - want).abs() / want.abs().clamp_min(want.pow(2).mean().sqrt() + 1e-30)
    assert float(err.max()) <= tol, float(err.max())


def inputs(rows, d, f, gathered, matrices):
    g = torch.Generator().manual_seed(sum(rows) + d + 3 * f)
    E, B = len(rows), sum(rows)
    off = torch.tensor([0] + list(torch.tensor(rows).cumsum(0)), dtype=torch.int32)
    T = 37 if gathered else B
    x = torch.randn((T, d), generator=g).bfloat16()
    index = torch.randint(0, T, (B,), generator=g, dtype=torch.int32) if gathered else None
    w = [(torch.randn((E, f, d) if i == matrices - 1 else (E, d, f), generator=g) * 0.05).bfloat16()
         for i in range(matrices)]
    xs = x[index.long()] if gathered else x
    return x, xs, index, off, w


@pytest.mark.parametrize("gathered", [False, True])
@pytest.mark.parametrize("d,f", WIDTHS)
@pytest.mark.parametrize("rows", ROWS, ids=list(ROWS))
def test_swiglu(rows, d, f, gathered):
    import paper_2508_13337_amd as m
    rows = ROWS[rows]
    x, xs, index, off, (wg, wu, wd) = inputs(rows, d, f, gathered, 3)
    E, B = len(rows), sum(rows)
    act = dict(dtype=torch.bfloat16, device="cuda")
    G, U, Y = torch.full((B + 1, f), 7.0, **act), torch.full((B + 1, f), 7.0, **act), torch.full((B + 1, d), 7.0, **act)
    ws = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_FFN_FWD, B, d, E, 1, f, m.XMOE_BF16))
    m.xmoe_expert_ffn_fwd(x.cuda(), off.cuda(), wg.cuda(), wu.cuda(), wd.cuda(), G[:B], U[:B], Y[:B], ws,
                          row_index=None if index is None else index.cuda())
    G, U, Y = G.cpu(), U.cpu(), Y.cpu()
    for o in (G, U, Y):
        assert bool((o[B] == 7.0).all())
    for e in range(E):
        s = slice(int(off[e]), int(off[e + 1]))
        if rows[e] == 0:
            continue
        g64, u64 = xs[s].double() @ wg[e].double(), xs[s].double() @ wu[e].double()
        close(G[s], g64)
        close(U[s], u64)
        a = g64 * torch.sigmoid(g64) * u64
        # A is rounded to bf16 in between: one rounding more, averaged over f terms
        close(Y[s], a.bfloat16().double() @ wd[e].double(), 2.0 ** -6)


@pytest.mark.parametrize("act", ["identity", "gelu", "silu"])
@pytest.mark.parametrize("d,f", [(64, 64), (192, 448)])
def test_two_matrix(d, f, act):
    import paper_2508_13337_amd as m
    rows = ROWS["edges"]
    x, xs, index, off, (w1, w2) = inputs(rows, d, f, True, 2)
    E, B = len(rows), sum(rows)
    t = dict(dtype=torch.bfloat16, device="cuda")
    H, Y = torch.empty((B, f), **t), torch.empty((B, d), **t)
    ws = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_MLP2_FWD, B, d, E, 1, f, m.XMOE_BF16))
    m.xmoe_expert_mlp2_fwd(x.cuda(), off.cuda(), w1.cuda(), w2.cuda(), act, H, Y, ws, row_index=index.cuda())
    H, Y = H.cpu(), Y.cpu()
    for e in range(E):
        s = slice(int(off[e]), int(off[e + 1]))
        if rows[e] == 0:
            continue
        h = xs[s].double() @ w1[e].double()
        close(H[s], h)
        a = {"identity": h, "gelu": torch.nn.functional.gelu(h), "silu": h * torch.sigmoid(h)}[act]
        close(Y[s], a.bfloat16().double() @ w2[e].double(), 2.0 ** -6)
