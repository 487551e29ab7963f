"""Forward products of experts with few rows (xmoe_ffn_few.hip, taken up to 32 rows per expert on average): segments at
the edges of a 32- and a 64-row block, several row tiles per expert, empty experts, widths of one and of several
64-column tiles.  Every test asserts the kernels that ran.

Tolerance: G, U, H and the activations are one float32-accumulated product rounded to bf16 (2^-9 relative) against a
float64 product of the same operands; an element that cancels to below the RMS is held to that share of the RMS."""
import pytest
import torch

from gpu_util import launched

pytestmark = pytest.mark.gpu

# the empty experts behind each list keep the mean within the rule
ROWS = {
    "edges": [0, 1, 31, 32, 33, 63, 64, 65, 0] + [0] * 10,      # 289 rows, 19 experts
    "one long": [1, 0, 200, 0, 3, 0] + [0] * 7,                 # 204 rows, 13 experts: four row tiles of one expert
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


def swiglu(m, x, off, w, B, index=None):
    """(G, U, Y, kernels) of one call; a marked row behind each output has to stand."""
    E, d, f = w[0].shape
    act = dict(dtype=torch.bfloat16, device="cuda")
    o = [torch.full((B + 1, n), 7.0, **act) for n in (f, f, d)]
    ws = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_FFN_FWD, B, d, E, 1, f, m.XMOE_BF16))
    args = (x.cuda(), off.cuda(), *(a.cuda() for a in w), *(t[:B] for t in o), ws)
    kernels = launched(m, lambda: m.xmoe_expert_ffn_fwd(*args, row_index=None if index is None else index.cuda()))
    o = [t.cpu() for t in o]
    assert all(bool((t[B] == 7.0).all()) for t in o)
    return [t[:B] for t in o] + [kernels]


def mlp2(m, x, off, w, act, B, index=None):
    E, d, f = w[0].shape
    o = [torch.full((B + 1, n), 7.0, dtype=torch.bfloat16, device="cuda") for n in (f, d)]
    ws = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_MLP2_FWD, B, d, E, 1, f, m.XMOE_BF16))
    args = (x.cuda(), off.cuda(), *(a.cuda() for a in w), act, *(t[:B] for t in o), ws)
    kernels = launched(m, lambda: m.xmoe_expert_mlp2_fwd(*args, row_index=None if index is None else index.cuda()))
    o = [t.cpu() for t in o]
    assert all(bool((t[B] == 7.0).all()) for t in o)
    return [t[:B] for t in o] + [kernels]


@pytest.mark.parametrize("gathered", [False, True])
@pytest.mark.parametrize("d,f", WIDTHS)
@pytest.mark.parametrize("rows", ROWS, ids=list(ROWS))
def test_swiglu(rows, d, f, gathered):
    import paper_2508_13337_amd as m
    rows = ROWS[rows]
    x, xs, index, off, w = inputs(rows, d, f, gathered, 3)
    G, U, Y, kernels = swiglu(m, x, off, w, sum(rows), index)
    assert kernels == {"tile_map_kernel", "ffn_gateup_few_kernel", "ffn_down_few_kernel"}, kernels
    for e in range(len(rows)):
        s = slice(int(off[e]), int(off[e + 1]))
        if rows[e] == 0:
            continue
        g64, u64 = xs[s].double() @ w[0][e].double(), xs[s].double() @ w[1][e].double()
        close(G[s], g64)
        close(U[s], u64)
        a = g64 * torch.sigmoid(g64) * u64
        # A is rounded to bf16 in between: one rounding more, averaged over f terms
        close(Y[s], a.bfloat16().double() @ w[2][e].double(), 2.0 ** -6)


@pytest.mark.parametrize("act", ["identity", "gelu", "silu"])
@pytest.mark.parametrize("d,f", [(64, 64), (192, 448)])
@pytest.mark.parametrize("rows", ["edges", "one long"])
def test_two_matrix(rows, d, f, act):
    import paper_2508_13337_amd as m
    rows = ROWS[rows]
    x, xs, index, off, w = inputs(rows, d, f, True, 2)
    H, Y, kernels = mlp2(m, x, off, w, act, sum(rows), index)
    assert kernels == {"tile_map_kernel", "mlp2_up_few_kernel", "ffn_down_few_kernel"}, kernels
    for e in range(len(rows)):
        s = slice(int(off[e]), int(off[e + 1]))
        if rows[e] == 0:
            continue
        h = xs[s].double() @ w[0][e].double()
        close(H[s], h)
        a = {"identity": h, "gelu": torch.nn.functional.gelu(h), "silu": h * torch.sigmoid(h)}[act]
        close(Y[s], a.bfloat16().double() @ w[1][e].double(), 2.0 ** -6)


@pytest.mark.parametrize("expert", ["swiglu", "identity", "gelu", "silu"])
@pytest.mark.parametrize("d,f", [(64, 64), (320, 192), (2048, 1408)])
def test_a_rows_bits_do_not_depend_on_the_row_count(d, f, expert):
    """The same tokens in a call with few rows and among many others (a decoding step, and a prompt, of one sequence):
    the direct-to-LDS kernels and these give the same bits, since both add K's products in one ascending order."""
    import paper_2508_13337_amd as m
    few, extra = [1, 0, 33, 64, 7] + [0] * 8, [40, 3, 300, 70, 1] + [100] * 8
    x, _, index, off, w = inputs(few, d, f, True, 3 if expert == "swiglu" else 2)
    g = torch.Generator().manual_seed(d)
    many = [a + b for a, b in zip(few, extra)]
    parts = []
    for e, n in enumerate(extra):     # every expert's rows of the small call, then others
        parts += [index[int(off[e]):int(off[e + 1])], torch.randint(0, 37, (n,), generator=g, dtype=torch.int32)]
    off2 = torch.tensor([0] + list(torch.tensor(many).cumsum(0)), dtype=torch.int32)
    call = (lambda *a: swiglu(m, *a)) if expert == "swiglu" else (lambda x, o, w, B, i: mlp2(m, x, o, w, expert, B, i))
    a = call(x, off, w, sum(few), index)
    b = call(x, off2, w, sum(many), torch.cat(parts))
    assert any("_few_" in k for k in a[-1]) and not any("_few_" in k for k in b[-1]), (a[-1], b[-1])
    for p, q in zip(a[:-1], b[:-1]):
        for e, n in enumerate(few):
            assert torch.equal(p[int(off[e]):int(off[e]) + n], q[int(off2[e]):int(off2[e]) + n]), (expert, e)


@pytest.mark.parametrize("E,f,rows,few", [(256, 64, 8192, True), (256, 64, 8193, False), (4, 192, 128, True),
                                          (4, 192, 129, False)])
def test_both_sides_of_the_rule(E, f, rows, few):
    import paper_2508_13337_amd as m
    d = 64
    count = [rows // E + (e < rows % E) for e in range(E)]
    x, xs, index, off, w = inputs(count, d, f, True, 2)
    H, Y, kernels = mlp2(m, x, off, w, "identity", rows, index)
    assert ("mlp2_up_few_kernel" in kernels) == few and ("mlp2_up_dma_kernel" in kernels) != few, kernels
    e = torch.repeat_interleave(torch.arange(E), torch.tensor(count))
    close(H, torch.bmm(xs.float().unsqueeze(1), w[0].float()[e]).squeeze(1).double())
