"""Router logits bit for bit against the oracle's fused-multiply-add chain, at
sizes that take each block tile of the logits kernel (one token past a whole
number of blocks, partial last chunks of the hidden index, expert counts that
are and are not multiples of four)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [(1, 8, 1), (17, 136, 33), (70, 264, 1000),   # one 16 x 16 tile per block
         (4129, 40, 20),                              # 32 x 32
         (16385, 24, 50),                             # 32 x 64
         (32769, 72, 62),                             # 64 x 64
         (32769, 40, 120),                            # 64 x 128
         (65537, 24, 126)]                            # 128 x 128


@pytest.mark.parametrize("T,d,E", SIZES)
def test_logits_bit_exact(T, d, E):
    from paper_2607_01844_amd import moe
    print(f"[route tiles] T={T} d={d} E={E}", flush=True)
    gen = torch.Generator().manual_seed(T + E)
    x = torch.randn((T, d), generator=gen).to(torch.bfloat16)
    # a wide spread of exponents: sums that round at every step
    w = torch.randn((d, E), generator=gen) * torch.exp2(
        torch.randint(-12, 12, (d, E), generator=gen).float())
    bias = torch.randn((E,), generator=gen) if E % 2 else None
    k = min(2, E)
    logits = torch.full((T, E), float("nan"), device="cuda")
    idx, _ = moe.moe_route(x.cuda(), w.cuda(), None if bias is None else bias.cuda(), k,
                           logits=logits)
    ref = oracle.logits(W.bf16_bits(x), w.numpy(), None if bias is None else bias.numpy(), "f32")
    assert np.array_equal(logits.cpu().numpy().view(np.int32), ref.view(np.int32))
    assert np.array_equal(idx.cpu().numpy(), oracle.topk(ref, k, 0)[0])
