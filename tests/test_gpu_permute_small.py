"""The permutation around the line between its one-launch form (up to 8192
assignments of up to 512 experts) and the three-launch form, against the
stable counting sort: expert ranges, uneven loads, counts of all experts, and
expert ids no rank holds (their assignments get no row)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [  # T, E, k, expert_begin, num_local
    (1, 1, 1, 0, 1), (3, 7, 2, 2, 3), (1023, 5, 1, 0, 5), (1024, 16, 4, 3, 9),
    (2048, 64, 4, 0, 64), (2049, 64, 4, 0, 64), (4096, 512, 2, 100, 300), (4097, 512, 2, 0, 512),
    (512, 513, 16, 0, 513), (8192, 2, 1, 1, 1),
]


@pytest.mark.parametrize("T,E,k,begin,local", CASES)
@pytest.mark.parametrize("skew", [0.0, 3.0])
def test_permutation(T, E, k, begin, local, skew):
    from paper_2607_01844_amd import moe
    print(f"[permute small] T={T} E={E} k={k} local=[{begin}, {begin + local}) skew={skew}",
          flush=True)
    rng = np.random.default_rng(T + E)
    logp = -skew * np.log(np.arange(1, E + 1))
    idx = np.argsort(-(logp + rng.gumbel(size=(T, E))), axis=1)[:, :k].astype(np.int32)
    d = 72
    x = torch.randn((T, d), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16).cuda()
    out = moe.moe_permute(x, torch.from_numpy(idx).cuda(), E, begin, local)
    flat = idx.ravel()
    a = np.nonzero((flat >= begin) & (flat < begin + local))[0]
    src = a[np.argsort(flat[a], kind="stable")]
    dst = np.full(T * k, -1, np.int32)
    dst[src] = np.arange(src.size)
    n = np.bincount(flat, minlength=E)
    off = np.concatenate([[0], np.cumsum(n[begin:begin + local])])
    M = src.size
    assert np.array_equal(out["expert_offsets"].cpu().numpy(), off)
    assert np.array_equal(out["counts_global"].cpu().numpy(), n)
    assert np.array_equal(out["dst"].cpu().numpy().ravel(), dst)
    assert np.array_equal(out["row_src"].cpu().numpy()[:M], src)
    tok = torch.from_numpy(src // k).cuda()
    assert torch.equal(out["x_perm"][:M].view(torch.int16), x[tok].view(torch.int16))
