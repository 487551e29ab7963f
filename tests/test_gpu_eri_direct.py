"""xmoe_build_eri on either side of the line between its one-launch and its three-launch construction (16 chunks of
1024 flat entries), with chunks that are not full, expert counts up to the limit and loads that all fall on the same
few experts (the counters are kept in several copies from 5 chunks on): bit-equal to a stable sort."""
import pytest
import torch

from gpu_util import launched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("load", ["even", "same experts"])
@pytest.mark.parametrize("T,E,k", [(1, 1, 1), (1, 512, 8), (170, 64, 6), (171, 64, 6), (2730, 64, 6), (2731, 64, 6),
                                   (2048, 512, 8), (2049, 512, 8), (16384, 7, 1), (333, 96, 3), (4096, 130, 1),
                                   (4097, 128, 1), (1366, 129, 3), (1400, 257, 6)])
def test_tables(T, E, k, load):
    import paper_2508_13337_amd as m
    g = torch.Generator().manual_seed(T + E + k)
    idx = torch.rand((T, E), generator=g).argsort(1)[:, :k].int().contiguous()
    if load == "same experts":
        idx = idx[:1].repeat(T, 1)
    w = torch.rand((T, k), generator=g)
    B = T * k
    i32 = dict(dtype=torch.int32, device="cuda")
    tpe, off = torch.full((E,), -9, **i32), torch.full((E + 1,), -9, **i32)
    tok, exp, row = (torch.full((B,), -9, **i32) for _ in range(3))
    cw = torch.empty(B, dtype=torch.float32, device="cuda")
    ws = m.alloc_workspace(m.xmoe_workspace_bytes(m.WS_BUILD_ERI, T, 64, E, k, 0, m.XMOE_BF16))
    kernels = launched(m, lambda: m.xmoe_build_eri(idx.cuda(), w.cuda(), E, tpe, off, tok, exp, cw, row, ws))
    assert kernels == ({"eri_direct_kernel"} if B <= 16 * 1024 else
                       {"eri_hist_kernel", "eri_scan_kernel", "eri_scatter_kernel"}), kernels
    flat = idx.reshape(-1).long()
    order = torch.sort(flat, stable=True).indices
    count = torch.bincount(flat, minlength=E)
    inverse = torch.empty(B, dtype=torch.long)
    inverse[order] = torch.arange(B)
    for got, want in ((tpe, count), (off[1:], count.cumsum(0)), (tok, order // k), (exp, flat[order]), (row, inverse)):
        assert torch.equal(got.cpu().long(), want)
    assert int(off[0]) == 0
    assert torch.equal(cw.cpu(), w.reshape(-1)[order])
