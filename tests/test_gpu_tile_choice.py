"""Row tiles that the device chooses by the experts' rows (e4m3 weights): each choice at sizes
where it is made, read back from the tile tables, and the outputs against the same products in
64 bits."""
import numpy as np
import pytest
import torch

import paper_2601_08800_amd as moe
from paper_2601_08800_amd.layer import config_from_workload
from test_gpu_fp8act import BASE

pytestmark = pytest.mark.gpu

SHORT, COUNT = 1 << 30, (1 << 29) - 1      # first word of a table: flag of the short tiles, their number


def _align(v):
    return (v + 255) // 256 * 256


def _weights(g, n, rows, cols):
    """Codes of N(0, 0.02) weights, block scales a factor of two apart on average from one K block
    to the next (a scale of the wrong block shows), and the values they stand for."""
    w = torch.empty(n, rows, cols, device="cuda").normal_(0, 0.02, generator=g)
    b = w.view(n, rows // 128, 128, cols // 128, 128)
    b *= torch.exp2(torch.empty(n, rows // 128, 1, cols // 128, 1, device="cuda").uniform_(-1, 1, generator=g))
    s = b.abs().amax(dim=(2, 4)) / 448
    q = (b / s[:, :, None, :, None]).to(torch.float8_e4m3fn)
    return (q.view(torch.uint8).view(n, rows, cols).contiguous(), s.contiguous(),
            lambda e: (q[e].double() * s[e].double()[:, None, :, None]).view(rows, cols))


def _quantised(v):
    r, k = v.shape
    b = v.float().view(r, k // 128, 128)
    s = b.abs().amax(2) / 448
    s = torch.where(s > 0, s, torch.ones_like(s))
    q = (b / s[:, :, None]).clamp(-448, 448).to(torch.float8_e4m3fn)
    return (q.double() * s.double()[:, :, None]).view(r, k)


def run_ffn(counts, H, I, fp8_acts=False, loose=1, row_scale=None):
    """One expert-FFN call on rows of given experts; returns (outputs, 64-bit reference, workspace)."""
    n, rows = len(counts), int(sum(counts))
    g = torch.Generator(device="cuda").manual_seed(H + I + rows)
    cfg = config_from_workload(BASE.replace(name="tile_choice", H=H, I=I, E=n, k=1, expert_lo=0, expert_hi=n))
    x = torch.empty(rows * loose, H, device="cuda").normal_(0, 1, generator=g)
    if row_scale is not None:
        x *= torch.tensor(row_scale, device="cuda")[torch.arange(len(x), device="cuda") % len(row_scale), None]
    x = x.bfloat16()
    (wg, sg, dg), (wu, su, du), (wd, sd, dd) = (_weights(g, n, *s) for s in ((I, H), (I, H), (H, I)))
    ends = np.concatenate([[0], np.cumsum(counts)])
    offsets = torch.tensor(ends, dtype=torch.int32, device="cuda")
    ys = torch.full((rows * loose, H), 7.0, device="cuda", dtype=torch.bfloat16)
    need = moe.moe_fp8act_workspace_bytes(cfg, n, rows * loose) if fp8_acts else moe.moe_workspace_bytes(cfg, rows * loose)
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    call = moe.moe_expert_ffn_fp8act if fp8_acts else moe.moe_expert_ffn
    call(cfg, n, x, offsets, rows * loose, wg, wu, wd, sg, su, sd, ys, ws)
    first = ys.clone()
    call(cfg, n, x, offsets, rows * loose, wg, wu, wd, sg, su, sd, ys, ws)
    assert torch.equal(first, ys), "not the same bits twice"
    assert bool((ys[rows:] == 7.0).all()), "rows past the last valid one were written"
    ref = torch.empty(rows, H, dtype=torch.float64, device="cuda")
    xv = _quantised(x[:rows]) if fp8_acts else x[:rows].double()
    for e in range(n):
        lo, hi = int(ends[e]), int(ends[e + 1])
        if lo == hi:
            continue
        a = xv[lo:hi] @ dg(e).t().contiguous()
        h = a * torch.sigmoid(a) * (xv[lo:hi] @ du(e).t().contiguous())
        if fp8_acts:
            h = _quantised(h)
        ref[lo:hi] = h @ dd(e).t().contiguous()
    return ys[:rows].double(), ref, ws


def check(got, ref, rel, largest):
    err = float((got - ref).norm() / ref.norm())
    worst = float((got - ref).abs().max() / ref.abs().max())
    print("rel %.3e max %.3e" % (err, worst), flush=True)
    assert err <= rel and worst <= largest


def tables(ws, rows, n):
    """Per GEMM: (short tiles?, tallest tile)."""
    words = ws.cpu().numpy().view(np.int32)
    out = []
    for at in (0, _align((1 + 5 * (rows // 32 + n + 1)) * 4 + 12) // 4):
        count = int(words[at]) & COUNT
        rec = words[at + 1:at + 1 + 5 * count].reshape(count, 5)
        out.append((bool(words[at] & SHORT), int((rec[:, 2] - rec[:, 1]).max())))
    return out


# bf16 activations, outputs and intermediate (2^-9 each, rounded) and code * scale rounded to
# bf16 where tiles are not short: about 4e-3 together; the layer's bar for the largest difference.
@pytest.mark.parametrize("counts,H,I,loose,want", [
    # one round of 64-row tiles in both GEMMs (8 column tiles each)
    ([40] * 31 + [64], 2048, 1024, 1, [64, 64]),
    # one expert of 90: another 64-row tile would open a second round of GEMM-1, 96 rows do not
    ([40] * 31 + [90], 128, 1024, 1, [96, 64]),
    # ... of 97: 128 rows; of 161, the capacity loose: a tall tile of 161 rows
    ([40] * 31 + [97], 128, 1024, 8, [128, 64]),
    ([40] * 31 + [161], 128, 1024, 8, [None, 64]),
    # the same choices in GEMM-2
    ([20] * 31 + [90], 2048, 128, 1, [64, 96]),
    ([20] * 30 + [200], 2048, 128, 1, [64, 128]),
    # a quarter of a round more against tall tiles of 185 rows (K split of the 48 left over)
    ([40] * 28 + [100, 120, 126, 185], 6144, 1024, 8, [64, 64]),
    # long groups, tight and loose capacity
    ([200] * 32, 128, 1024, 1, [None, 64]),
    ([200] * 32, 128, 1024, 4, [None, 64]),
    # against the wide tiles of GEMM-2: 64 and 80 experts x 8 column tiles, 4 counted double
    ([13] * 64, 2048, 128, 1, [64, None]),
    ([13] * 80, 2048, 128, 1, [64, 64]),
    # leftover tiles cut along K: 33 experts x 8 column tiles, 26 K blocks in two parts
    ([20] * 33, 3328, 1024, 1, [64, 64]),
    # a single expert of 12 x 8, 12 x 8 and 20 x 8 whole tiles; of 11 x 8 and 21 x 8
    ([1409], 128, 1024, 1, [128, None]),
    ([1531], 3328, 1024, 1, [128, None]),
    ([2560], 128, 1024, 1, [128, None]),
    ([1408], 128, 1024, 1, [None, None]),
    ([2561], 128, 1024, 1, [None, None]),
    # empty first and last experts, one-row experts
    ([0, 1, 31, 32, 33, 64, 0, 1, 63, 2, 0], 256, 384, 2, [64, 64])],
    ids=lambda v: "%dx%d" % (len(v), max(c or 0 for c in v)) if isinstance(v, list) else str(v))
def test_e4m3_tiles(counts, H, I, loose, want):
    got, ref, ws = run_ffn(counts, H, I, loose=loose)
    check(got, ref, 1.5e-2, 6e-2)
    for (short, tallest), height in zip(tables(ws, sum(counts) * loose, len(counts)), want):
        assert short == (height is not None), (short, tallest)
        assert height is None or tallest <= height


# K past 64 blocks of 128: each GEMM loads its block scales again at block 64.  e4m3 weights on short
# tiles, GEMM-1 (one expert, 98 tiles) and GEMM-2 (80 experts, 4 column tiles), and on tall tiles
# of few rows, cut along K; 8-bit activations with one, two and six row blocks a tile.
@pytest.mark.parametrize("counts,H,I,want", [
    ([12544], 8448, 128, [128, None]), ([14] * 80, 1024, 8448, [64, 64]),
    ([40, 17], 8448, 128, [None, 64]), ([40, 17], 128, 8448, [64, None])],
    ids=lambda v: str(v) if isinstance(v, int) else "")
def test_e4m3_scales_past_64_blocks(counts, H, I, want):
    got, ref, ws = run_ffn(counts, H, I)
    check(got, ref, 1.5e-2, 6e-2)
    for (short, _), height in zip(tables(ws, sum(counts), len(counts)), want):
        assert short == (height is not None)


@pytest.mark.parametrize("counts,H,I", [([33, 1, 64], 8320, 128), ([40, 192], 256, 8448), ([5], 16512, 128)])
def test_fp8act_scales_past_64_blocks(counts, H, I):
    got, ref, _ = run_ffn(counts, H, I, fp8_acts=True)
    check(got, ref, 1.5e-2, 6e-2)


# Intermediates past 2^90 and below 2^-90 take the quantiser's general division, all 32 rows of a
# block or some of them; every row is compared at its own magnitude.
@pytest.mark.parametrize("row_scale", [[2.0**50], [2.0**-50], [1.0, 2.0**50, 2.0**-50, 2.0**20]])
def test_fp8act_quotients_near_the_ends_of_the_range(row_scale):
    got, ref, _ = run_ffn([40, 0, 200, 31], 256, 256, fp8_acts=True, row_scale=row_scale)
    norm = ref.abs().amax(1, keepdim=True)
    assert bool((norm > 0).all())
    check(got / norm, ref / norm, 1.5e-2, 6e-2)
