"""Router logits bit for bit against the oracle's fused-multiply-add chain, at
sizes that take each block tile of the logits kernel: one token past a whole
number of blocks, expert counts that are and are not multiples of four (16- and
4-byte weight loads), and hidden sizes of less than a chunk and of two chunks
more than the LDS ring holds and a partial one.  And operands and logits that
are not ordinary numbers."""
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
# (ring slots + 2) chunks of KC hidden indices and 8 more
SIZES += [(17, 6 * 128 + 8, 33), (17, 6 * 128 + 8, 36), (4129, 6 * 64 + 8, 18), (4129, 6 * 64 + 8, 20),
          (16385, 6 * 64 + 8, 50), (16385, 6 * 64 + 8, 52), (32769, 5 * 64 + 8, 62),
          (32769, 5 * 64 + 8, 60), (32769, 6 * 32 + 8, 118), (32769, 6 * 32 + 8, 120),
          (65537, 5 * 32 + 8, 126), (65537, 5 * 32 + 8, 124)]


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


@pytest.mark.parametrize("T", [40, 4129])   # one wave a block, four waves a block
@pytest.mark.parametrize("E", [20, 22])
def test_special_values(T, E):
    """Subnormal operands, products and sums, signed zeros, infinities and NaN
    through the matrix instruction: NaN where the chain has NaN, every other
    bit the chain's; then the selection: NaN ranks as -inf, equal logits (-0
    and +0 among them, and rows that are all -inf) go to the lower index."""
    from paper_2607_01844_amd import moe
    print(f"[route special] T={T} E={E}", flush=True)
    d, k = 136, 6
    gen = torch.Generator().manual_seed(T + E)
    x = torch.randn((T, d), generator=gen)
    w = torch.randn((d, E), generator=gen)
    kind = torch.arange(T) % 8
    x[kind == 1] *= 2.0 ** -70                 # with the small columns: subnormal products
    x[kind == 2] *= 2.0 ** -130                # subnormal operands
    x[kind == 3] *= 2.0 ** -100                # sums that round to a signed zero
    x[kind == 4] = torch.where(torch.rand((int((kind == 4).sum()), d), generator=gen) < 0.5, 0.0, -0.0)
    x[kind == 5, 3] = float("inf")             # inf, and inf * 0 = NaN
    x[kind == 6, 5] = float("inf")             # inf - inf = NaN in some columns
    x[kind == 6, 7] = float("-inf")
    x[kind == 7, 9] = float("nan")             # NaN everywhere
    w[:, 0:4] *= 2.0 ** -70
    w[:, 4:6] *= 2.0 ** -128                   # subnormal weights
    w[:, 6:8] *= 2.0 ** -100
    w[:, 8] = 0.0
    w[:, 9] = -0.0
    w[3, 10] = 0.0
    w[11, 11] = float("inf")
    w[12, 12] = float("-inf")
    # one token's row ends in a product that underflows: a logit of -0
    x[3], w[:, 6], w[:, 7] = 0.0, 0.0, 0.0
    x[3, d - 1], w[d - 1, 6], w[d - 1, 7] = -2.0 ** -100, 2.0 ** -100, -2.0 ** -100
    xb = x.to(torch.bfloat16)
    bias = torch.zeros((E,))
    bias[13:15] = float("-inf")
    for b in (None, bias):
        logits = torch.full((T, E), 7.0, device="cuda")
        idx, _ = moe.moe_route(xb.cuda(), w.cuda(), None if b is None else b.cuda(), k, logits=logits)
        ref = oracle.logits(W.bf16_bits(xb), w.numpy(), None if b is None else b.numpy(), "f32")
        got, nan = logits.cpu().numpy(), np.isnan(ref)
        assert np.array_equal(np.isnan(got), nan)
        assert np.array_equal(got.view(np.int32)[~nan], ref.view(np.int32)[~nan])
        assert np.array_equal(idx.cpu().numpy(), oracle.topk(ref, k, 0)[0])
        if b is None:  # the cases are there
            sub = (ref != 0) & (np.abs(ref) < 2.0 ** -126)
            assert sub.any() and nan.any() and np.isinf(ref).any()
            assert ref.view(np.uint32)[3, 6] == 0x80000000 and ref.view(np.uint32)[3, 7] == 0
    # every logit -inf: the lowest indices in order
    idx, _ = moe.moe_route(xb.cuda(), w.cuda(), torch.full((E,), float("-inf"), device="cuda"), k)
    assert torch.equal(idx[0].cpu(), torch.arange(k, dtype=torch.int32))
