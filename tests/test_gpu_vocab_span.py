"""Vocabulary loss where every product of its first block takes the 256-row
tile, and dW the ping-pong schedule, with rows of W and dW of every alignment, and the forward
over one block at a time (a workspace that holds the forward's buffers only)
bit for bit against the forward over many."""
import ctypes

import pytest
import torch

import workloads as W
from tests import parity as P

pytestmark = pytest.mark.gpu


def _inputs(N, H, V, seed):
    return W.make_vocab_inputs(W.VocabWorkload("case", N=N, H=H, V=V, vblock=8), seed=seed,
                               device="cuda")


@pytest.mark.parametrize("V", [17003, 17000, 16390])
def test_large_tiles_any_row_alignment(V):
    from paper_2607_01844_amd import moe
    N, H, vb = 2040, 1000, 16384
    rows, cols = 8, 4  # 256-row tiles over N and H
    assert P.large_tile(rows * -(-V // 256))       # forward (all of V at once)
    assert P.large_tile(rows * (vb // 256))        # logit gradients
    assert P.large_tile(8 * rows * cols)           # dx, in 8 ranges of the block
    assert P.large_tile(cols * (vb // 256)) and N >= 16 * 64  # dW, ping-pong
    print(f"[vocab span] N={N} H={H} V={V}", flush=True)
    i = _inputs(N, H, V, V)
    dw = torch.full((H, V), float("nan"), dtype=torch.bfloat16, device="cuda")
    loss, lse = moe.moe_vocab_loss_fwd(i["x"], i["w_voc"], i["target"], vb)
    dx, dw = moe.moe_vocab_loss_bwd(i["x"], i["w_voc"], i["target"], lse, i["dloss"], vb, dw_voc=dw)
    x, w, t = i["x"].double(), i["w_voc"].double(), i["target"].long()
    y = x @ w
    ref_lse = torch.logsumexp(y, 1)
    G = -torch.exp(y - ref_lse[:, None])
    G[torch.arange(N, device="cuda"), t] += 1.0
    G *= i["dloss"].double()[:, None]
    P.assert_close("lse", P.f64(lse), ref_lse.cpu().numpy(), 1e-5)
    P.assert_close("loss", P.f64(loss), (y.gather(1, t[:, None])[:, 0] - ref_lse).cpu().numpy(), 1e-5)
    P.assert_close("dx", P.f64(dx), (G @ w.t()).cpu().numpy())
    P.assert_close("dw", P.f64(dw), (x.t() @ G).cpu().numpy())


# blocks of one to many groups of 64 columns, more than four blocks at once,
# a short last block, and blocks that end inside a group
@pytest.mark.parametrize("N,H,V,vb", [(70, 40, 1000, 64), (300, 24, 1001, 128), (70, 264, 9000, 1024),
                                      (33, 264, 40003, 8256), (70, 40, 1000, 104), (300, 24, 1001, 8)])
def test_forward_block_by_block_workspace(N, H, V, vb):
    from paper_2607_01844_amd import moe
    i = _inputs(N, H, V, 3)
    loss, lse = moe.moe_vocab_loss_fwd(i["x"], i["w_voc"], i["target"], vb)
    up = lambda v, a=256: (v + a - 1) // a * a  # noqa: E731
    need = up(8 * N * ((vb + 63) // 64)) + 3 * up(4 * N) + (up(2 * H * vb) if V % 8 else 0) + 256
    full = ctypes.c_size_t()
    assert moe.lib.moe_vocab_loss_workspace_bytes(N, H, V, vb, ctypes.byref(full)) == 0
    assert need < full.value
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    one = [torch.full((N,), float("nan"), device="cuda") for _ in range(2)]
    args = (i["x"].data_ptr(), i["w_voc"].data_ptr(), i["target"].data_ptr(), N, H, V, vb,
            one[0].data_ptr(), one[1].data_ptr(), ws.data_ptr())
    assert moe.lib.moe_vocab_loss_fwd(*args, need - 1, None) != 0  # still refused
    assert moe.lib.moe_vocab_loss_fwd(*args, need, moe._stream()) == 0
    # the same pairs merged in the same order
    assert torch.equal(one[0].view(torch.int32), loss.view(torch.int32))
    assert torch.equal(one[1].view(torch.int32), lse.view(torch.int32))
