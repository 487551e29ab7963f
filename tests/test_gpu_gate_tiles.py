"""xmoe_gate_logits on the K = 1 matrix instructions: the same bits as the oracle's loop, at the edges of its two tile
sizes (16 x 16 up to 16 experts, and below 256 blocks of 32 x 32), of its stages and of 16-byte vectors in either operand."""
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
