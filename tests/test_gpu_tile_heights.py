"""Expert products at row counts around every tile height: an expert's rows
are cut into equal tiles of whole 32-row blocks, the two wave rows holding up
to four blocks each.  Forward, data and weight gradients against fp32 on the
CPU (bf16 operands, fp32 sums: max error within 1e-2 of the largest value,
as for the whole layer)."""
import numpy as np
import pytest
import torch

from tests import parity as P

pytestmark = pytest.mark.gpu

COUNTS = {
    "one_tile": [1, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 255, 256],
    "two_tiles": [257, 0, 288, 320, 321, 352, 384, 385, 416, 448, 480, 511, 512],
    "three_tiles": [513, 576, 577, 0, 0, 640, 672, 704, 767, 768, 769],
    # up to 63 experts the 128-row launches form their tables in registers
    "experts_62": [(7 * i) % 43 for i in range(62)],
    "experts_63": [0] + [(7 * i) % 43 for i in range(62)],
    "experts_64": [(7 * i) % 43 for i in range(63)] + [40],
    "experts_65": [(7 * i) % 43 for i in range(63)] + [0, 300],
    # few rows an expert: 128-row data gradients beside (d = 2056) a 256-row
    # gate/up weight gradient, both sides of the in-register tables
    "few_rows_60": [i % 9 for i in range(60)],
    "few_rows_70": [130] + [i % 9 for i in range(69)],
}


# the tiles of the forward's gate/up and down products and of the data
# gradients: the 128-row tile (few tiles in all), the 256-row tile (more than
# two tiles per compute unit; few rows stay on the 128-row tile), and the two
# mixed in one pass, where the forward's two tables of row tiles differ
CASES = [(n, 72, 136, "SSS") for n in COUNTS]
CASES += [(n, 264, 328, "LLS" if n.startswith("experts") else "SSS") for n in COUNTS]
CASES += [(n, 72, 5128, "SSS" if n.startswith("few") else "LLL") for n in COUNTS]
CASES += [("experts_62", 1032, 264, "LSS"), ("experts_63", 1032, 264, "LSS"),
          ("two_tiles", 2440, 840, "SLS"), ("few_rows_60", 2056, 384, "SSS"),
          ("few_rows_70", 2056, 384, "SSS")]


@pytest.mark.parametrize("name,d,f,tiles", CASES)
def test_rows_around_tile_heights(name, d, f, tiles):
    from paper_2607_01844_amd import moe
    counts = COUNTS[name]
    print(f"[tile heights] {name} d={d} f={f}", flush=True)
    E, M = len(counts), sum(counts)
    up = lambda a, b: -(-a // b)  # noqa: E731
    assert P.row_tiles(M, E, d, f) == tiles
    if (d, f) == (2056, 384):  # the gate/up weight gradient
        assert P.large_weights(*(E * up(d, m) * up(f, m // 2) for m in (256, 128)))
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    gen = torch.Generator().manual_seed(M + d)
    r = lambda *s, std=1.0: (torch.randn(s, generator=gen) * std).to(torch.bfloat16)  # noqa: E731
    x, dy = r(M, d), r(M, d)
    wg, wu, wd = r(E, d, f, std=0.05), r(E, d, f, std=0.05), r(E, f, d, std=0.05)
    g = {k: v.cuda() for k, v in dict(x=x, dy=dy, wg=wg, wu=wu, wd=wd).items()}
    o = torch.from_numpy(off).cuda()
    nan = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda")  # noqa: E731
    hg, hu, y = moe.moe_grouped_swiglu_fwd(g["x"], o, g["wg"], g["wu"], g["wd"], h_gate=nan(M, f),
                                           h_up=nan(M, f), y_perm=nan(M, d))
    dx, dwg, dwu, dwd = moe.moe_grouped_swiglu_bwd(
        g["dy"], g["x"], hg, hu, o, g["wg"], g["wu"], g["wd"], dx_perm=nan(M, d),
        dw_gate=nan(E, d, f), dw_up=nan(E, d, f), dw_down=nan(E, f, d))
    ref = {n: [] for n in ("hg", "hu", "y", "dx", "dwg", "dwu", "dwd")}
    for e in range(E):
        s = slice(int(off[e]), int(off[e + 1]))
        xe, dye, g_, u_, w_ = x[s].float(), dy[s].float(), wg[e].float(), wu[e].float(), wd[e].float()
        a, b = xe @ g_, xe @ u_
        sg = torch.sigmoid(a)
        act, da = a * sg * b, dye @ w_.t()
        dg, du = da * b * sg * (1 + a * (1 - sg)), da * a * sg
        for n, v in dict(hg=a, hu=b, y=act @ w_, dx=dg @ g_.t() + du @ u_.t(), dwg=xe.t() @ dg,
                         dwu=xe.t() @ du, dwd=act.t() @ dye).items():
            ref[n].append(v)
    for n, got in dict(hg=hg, hu=hu, y=y, dx=dx).items():
        P.assert_close(n, P.f64(got), torch.cat(ref[n]).numpy())
    for n, got in dict(dwg=dwg, dwu=dwu, dwd=dwd).items():
        P.assert_close(n, P.f64(got), torch.stack(ref[n]).numpy())
