"""xmoe_gate_logits on the K = 1 matrix instructions: the same bits as the oracle's loop, at the edges of its two tile
sizes (16 x 16 up to 16 experts, and below 256 blocks of 32 x 32), of its stages and of 16-byte vectors in either operand.
xmoe_gate_logits_bwd in float32, and in bf16 where an operand's rows are no whole vectors, against float64."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as oracle

pytestmark = pytest.mark.gpu

SHAPES = [  # T, d, E
    (1, 1, 1), (1, 64, 3), (15, 63, 7), (16, 65, 16), (17, 512, 17), (33, 1000, 64), (8, 2048, 64), (3, 129, 512),
    (4096, 64, 64), (4095, 130, 63), (8161, 257, 1), (513, 384, 512), (1100, 77, 250),
    (8200, 136, 4), (8193, 513, 16), (8200, 256, 17), (8200, 250, 24), (9000, 1032, 20),
]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,d,E", SHAPES)
def test_logits_are_the_oracles_bits(T, d, E, dtype):
    import paper_2508_13337_amd as m
    g = torch.Generator().manual_seed(T * 31 + d * 7 + E)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x, w = (torch.randn(s, generator=g).to(dt) for s in ((T, d), (d, E)))
    bias = torch.randn(E, generator=g) if E % 2 else None
    want = oracle.gate_logits_contract(x.float().numpy(), w.float().numpy(), None if bias is None else bias.numpy())
    # operands that start one element into their storage: the loads have the alignment of one element
    xs, ws = (torch.empty(t.numel() + 1, dtype=dt, device="cuda")[1:].view(t.shape).copy_(t) for t in (x, w))
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda")
    m.xmoe_gate_logits(xs, ws, None if bias is None else bias.cuda(), logits)
    np.testing.assert_array_equal(logits.cpu().numpy().view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("T,E", [(20, 40), (8192, 33)])
@pytest.mark.parametrize("special", ["subnormal", "negative zero", "infinity"])
def test_special_values(T, E, special):
    import paper_2508_13337_amd as m
    d = 67
    g = torch.Generator().manual_seed(T + E)
    x, w = torch.randn((T, d), generator=g), torch.randn((d, E), generator=g)
    if special == "subnormal":      # products and sums below the smallest normal float32
        x, w = x * 1e-20, w * 1e-20
    elif special == "negative zero":    # every product rounds to a zero of either sign
        x, w = x * 1e-30, w * 1e-30
    else:                           # one infinite logit row and column, no NaN
        x[3], w[:, 2] = x[3].abs(), w[:, 2].abs()
        x[3, d - 1] = float("inf")
        w[d - 1] = w[d - 1].abs()
    want = oracle.gate_logits_contract(x.numpy(), w.numpy(), None)
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda")
    m.xmoe_gate_logits(x.cuda(), w.cuda(), None, logits)
    np.testing.assert_array_equal(logits.cpu().numpy().view(np.uint32), want.view(np.uint32))


# dx takes 32, 64, 128 or 256 columns per wave (the more the blocks): 585, 520 (d no multiple of the columns) and 516
# blocks at the last three; E on both sides of a 64-expert chunk; odd and even d and E
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("T,d,E", [(1, 1, 1), (16, 63, 2), (17, 64, 3), (257, 130, 65), (300, 129, 128), (700, 66, 63),
                                   (8197, 520, 9), (16500, 501, 24), (16500, 1001, 66)])
def test_backward_any_shape(T, d, E, shift, dtype):
    import paper_2508_13337_amd as m
    g = torch.Generator().manual_seed(T * 31 + d * 7 + E)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x, w = (torch.randn(s, generator=g).to(dt) for s in ((T, d), (d, E)))
    dl = torch.randn((T, E), generator=g)
    # shift: operands that start one element into their storage
    xs, ws, ds = (torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[shift:shift + t.numel()].view(t.shape).copy_(t)
                  for t in (x, w, dl))
    dw, dx = torch.full((d + 1, E), 5.0, dtype=dt, device="cuda"), torch.full((T + 1, d), 5.0, dtype=dt, device="cuda")
    tmp = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_GATE_BWD, T, d, E, 1, 0, m.dtype_code(dt)))
    m.xmoe_gate_logits_bwd(xs, ws, ds, dw[:d], dx[:T], tmp)
    assert bool((dw[d] == 5.0).all()) and bool((dx[T] == 5.0).all())
    x64, w64, dl64 = x.double().cuda(), w.double().cuda(), dl.double().cuda()
    # products of n terms summed in float32: n 2^-24 of the sum of the magnitudes; the bf16 kernels drop 2^-17 of every
    # dlogits element; one rounding of the result
    u, split = (2.0 ** -24, 0.0) if dtype == "f32" else (2.0 ** -8, 2.0 ** -16)
    for got, a, b, n in ((dw[:d], x64.t(), dl64, T), (dx[:T], dl64, w64.t(), E)):
        want, mag = a @ b, a.abs() @ b.abs()
        over = (got.double() - want).abs() - ((n + 8) * 2.0 ** -24 + split) * mag * 1.01 - u * want.abs() - 1e-30
        assert bool((over <= 0).all()), float(over.max())
