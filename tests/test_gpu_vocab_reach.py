"""Vocabulary loss where a row of W (or of the logit gradients) is so long
that a tile's rows span more than the 2^31 bytes a buffer descriptor reaches:
rows that are copied block by block (V not a multiple of 8), rows that would
be read in place, and one block longer than the limit.  Loss and lse of every
token, dx in full and dW at sampled columns (the last ones included) against
fp32 products of the same bf16 operands."""
import pytest
import torch

from tests import parity as P

pytestmark = pytest.mark.gpu

CASES = [  # N, H, V, vblock
    (64, 32, 40_000_001, 20_000_000),   # several blocks copied at once by the forward
    (64, 32, 40_000_000, 8_000_000),    # rows read in place
    (300, 264, 9_000_008, 65_536),      # the dx product's rows of W
    (300, 16, 9_000_008, 9_000_008),    # and of logit gradients, in one block
]


@pytest.mark.parametrize("N,H,V,vb", CASES)
def test_long_rows(N, H, V, vb):
    from paper_2607_01844_amd import moe
    print(f"[vocab reach] N={N} H={H} V={V} vblock={vb}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn((N, H), generator=gen, device="cuda").to(torch.bfloat16)
    w = torch.empty((H, V), dtype=torch.bfloat16, device="cuda")
    for h in range(H):
        w[h] = 0.3 * torch.randn((V,), generator=gen, device="cuda")
    t = torch.randint(0, V, (N,), generator=gen, device="cuda", dtype=torch.int32)
    t[-1], t[0] = V - 1, 0
    dloss = torch.randn((N,), generator=gen, device="cuda")
    loss, lse = moe.moe_vocab_loss_fwd(x, w, t, vb)
    dw = torch.full((H, V), float("nan"), dtype=torch.bfloat16, device="cuda")
    dx, dw = moe.moe_vocab_loss_bwd(x, w, t, lse, dloss, vb, dw_voc=dw)
    torch.cuda.synchronize()

    step = 1 << 20
    xf = x.float()
    parts, yt = [], torch.zeros((N,), device="cuda")
    for b in range(0, V, step):
        y = xf @ w[:, b:b + step].float()
        parts.append(torch.logsumexp(y, 1).double())
        here = (t >= b) & (t < b + y.shape[1])
        yt[here] = y[here, (t[here] - b).long()]
    ref_lse = torch.logsumexp(torch.stack(parts), 0)
    P.assert_close("lse", P.f64(lse), P.f64(ref_lse), 1e-5)
    P.assert_close("loss", P.f64(loss), P.f64(yt.double() - ref_lse), 1e-5)
    ref_dx = torch.zeros((N, H), dtype=torch.float64, device="cuda")
    for b in range(0, V, step):
        wb = w[:, b:b + step].float()
        g = -torch.exp((xf @ wb) - ref_lse[:, None].float())
        here = ((t >= b) & (t < b + wb.shape[1])).nonzero()[:, 0]
        g[here, (t[here] - b).long()] += 1.0
        g *= dloss[:, None]
        ref_dx += (g @ wb.t()).double()
        # this block's dW: sampled columns, its ends and its targets
        c = torch.cat([torch.tensor([0, wb.shape[1] - 1], device="cuda"), (t[here] - b).long(),
                       torch.randint(0, wb.shape[1], (64,), generator=gen, device="cuda")])
        P.assert_close(f"dw from {b}", P.f64(dw[:, b + c]), P.f64(xf.t() @ g[:, c]))
    P.assert_close("dx", P.f64(dx), P.f64(ref_dx))
