"""Expert-FFN kernels at the sizes where their tiles, chunks and rings can go wrong:
remainders of every tile dimension, K shorter and longer than a ring, empty and
one-row experts; outputs against the oracle on every token, and twice the same bits."""
import numpy as np
import pytest
import torch

import oracle
from helpers import TOL, check_dispatch, dev, host, inputs, make_layer, rel_err
from test_gpu_parity import _forced_counts_case

pytestmark = pytest.mark.gpu


def check_ffn(counts, H, I, tol, **changes):
    w, ids, tw = _forced_counts_case(counts, H=H, I=I, seed=3)
    w = w.replace(name="ffn_edges", **changes)
    d = inputs(w)
    L = make_layer(w, d)
    x, forced = dev(d["x"]), (dev(ids), dev(tw))
    out = host(L.forward(x, forced)).copy()
    torch.cuda.synchronize()
    check_dispatch(L, ids, w, d["x"])
    ref, _ = oracle.layer_share(d["x"], ids, tw, w.expert_lo, w.e_hi, d["experts"], d["shared"],
                                fp8_activations=w.fp8_activations)
    err = rel_err(out, ref)
    print("counts", counts, "H", H, "I", I, "err %.3e" % err, flush=True)
    assert err <= tol
    again = host(L.forward(x, forced))
    torch.cuda.synchronize()
    assert np.array_equal(out, again)


# K chunks of 128 values, rings of three (gate|up) and four chunks, tiles of 32 rows
# x 32 columns.  The tolerance is the layer's fp32 bar: sums of K <= 1032 products in
# fp32, sqrt(K) * 2^-24 of the largest value in the mean, about 2e-6.
@pytest.mark.parametrize("H,I", [(8, 8), (136, 40), (384, 512), (520, 640), (1032, 264)])
def test_fp32_tiles(H, I):
    check_ffn([1, 31, 32, 33, 0, 70], H, I, TOL["f32"], act_dtype="f32", weight_dtype="f32", x_std=0.02)


# GEMM-2 with K = I up to 128: one to eight K sub-steps, the last one partly filled,
# column blocks of 128 with a remainder, fewer blocks than one, 32-row blocks of the
# 128-row tiles on both sides of a border.  bf16 bar of the layer.
@pytest.mark.parametrize("H,I", [(64, 8), (136, 16), (392, 40), (1032, 72), (520, 96), (256, 104), (8, 128)])
@pytest.mark.parametrize("counts", [[1, 31, 33, 0, 2], [127, 128, 129, 300]])
def test_bf16_short_k(counts, H, I):
    check_ffn(counts, H, I, TOL["bf16"])


# K that is no multiple of 64 on the tall-tile kernel: full tiles (alternating loop) and
# short ones (rotated loop) whose last step is partly filled, columns that end inside a
# 32-column block, fewer steps than the rings have stages, and leftover tiles split
# along a K that ends in a short step (49 steps of GEMM-1).
@pytest.mark.parametrize("counts,H,I", [([256, 520, 40], 328, 200), ([300, 257], 72, 136),
                                        ([512, 97], 1032, 264), ([300], 3080, 136)])
def test_bf16_ragged_k_tall_tiles(counts, H, I):
    check_ffn(counts, H, I, TOL["bf16"])


# K that is no multiple of 64 on the weight-streaming kernel (at most two rows per
# expert on average, and GEMM-2 at up to twelve).
@pytest.mark.parametrize("counts", [[1, 2, 0, 3], [9, 1, 14, 8]])
def test_bf16_ragged_k_weight_streaming(counts):
    check_ffn(counts, 328, 200, TOL["bf16"])


# SwiGLU where g * u is past the fp32 range and silu(g) is zero: g = -2^66, u = 2^66 have the
# intermediate 0, at sizes that are no multiple of 64, on every kernel of GEMM-1 (the average
# number of rows picks it) and on both row halves of a tile.
@pytest.mark.parametrize("H,I", [(328, 200), (520, 136), (72, 96)])
@pytest.mark.parametrize("rows", [2, 24, 300, 700])
def test_bf16_ragged_swiglu_of_large_values(rows, H, I):
    import paper_2601_08800_amd as moe
    cfg = moe.MoEConfig(hidden=H, n_experts=1, top_k=1, score_fn=moe.MOE_SCORE_SOFTMAX, renormalize=1, routed_scale=1.0,
                        n_groups=1, topk_groups=1, group_score_n=0, expert_lo=0, expert_hi=1, inter_local=I,
                        act_dtype=moe.MOE_BF16, weight_dtype=moe.MOE_BF16)
    bf = lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device="cuda")
    x, wg, wu, wd, ys = bf(rows, H), bf(1, I, H), bf(1, I, H), bf(1, H, I), bf(rows, H)
    x[:, 0] = 2.0 ** 33
    wg[:, :, 0], wu[:, :, 0] = -2.0 ** 33, 2.0 ** 33
    wd.fill_(1.0)
    offsets = torch.tensor([0, rows], dtype=torch.int32, device="cuda")
    ws = torch.empty(moe.moe_workspace_bytes(cfg, rows), dtype=torch.uint8, device="cuda")
    ys.fill_(1.0)
    moe.moe_expert_ffn(cfg, 1, x, offsets, rows, wg, wu, wd, None, None, None, ys, ws)
    assert torch.count_nonzero(ys).item() == 0 and not torch.isnan(ys).any()


# An infinite gate keeps silu(g) = g (inf) on every kernel of GEMM-1, beside finite values in
# the same tile; the intermediate is then inf, and so is every output of that row.
@pytest.mark.parametrize("rows", [2, 24, 300])
def test_bf16_ragged_swiglu_of_infinity(rows):
    import paper_2601_08800_amd as moe
    H, I = 72, 96
    cfg = moe.MoEConfig(hidden=H, n_experts=1, top_k=1, score_fn=moe.MOE_SCORE_SOFTMAX, renormalize=1, routed_scale=1.0,
                        n_groups=1, topk_groups=1, group_score_n=0, expert_lo=0, expert_hi=1, inter_local=I,
                        act_dtype=moe.MOE_BF16, weight_dtype=moe.MOE_BF16)
    full = lambda v, *s: torch.full(s, v, dtype=torch.bfloat16, device="cuda")
    x, wg, wu, wd, ys = full(0.0, rows, H), full(0.0, 1, I, H), full(0.0, 1, I, H), full(1.0, 1, H, I), full(0.0, rows, H)
    x[:, 0] = 1.0
    x[rows - 1, 0] = 2.0 ** 100
    wg[:, :, 0], wu[:, :, 0] = 2.0 ** 100, 1.0          # g = 2^100, and past the range in the last row
    offsets = torch.tensor([0, rows], dtype=torch.int32, device="cuda")
    ws = torch.empty(moe.moe_workspace_bytes(cfg, rows), dtype=torch.uint8, device="cuda")
    moe.moe_expert_ffn(cfg, 1, x, offsets, rows, wg, wu, wd, None, None, None, ys, ws)
    assert bool((ys[:-1].float() == 96 * 2.0 ** 100).all()) and bool(torch.isposinf(ys[-1].float()).all())


def _ffn(counts, H, I, act="bf16"):
    """moe_expert_ffn on groups of `counts` rows, and fp64 torch on the same stored values (a bf16
    layer's intermediate rounded to bf16 as it is stored)."""
    import paper_2601_08800_amd as moe
    n, R = len(counts), sum(counts)
    cfg = moe.MoEConfig(hidden=H, n_experts=n, top_k=1, score_fn=moe.MOE_SCORE_SOFTMAX, renormalize=1, routed_scale=1.0,
                        n_groups=1, topk_groups=1, group_score_n=0, expert_lo=0, expert_hi=n, inter_local=I,
                        act_dtype=moe.MOE_BF16 if act == "bf16" else moe.MOE_F32,
                        weight_dtype=moe.MOE_BF16 if act == "bf16" else moe.MOE_F32)
    dt, bits = (torch.bfloat16, torch.int16) if act == "bf16" else (torch.float32, torch.int32)
    g = torch.Generator(device="cuda").manual_seed(R + H + I)
    draw = lambda std, *s: torch.empty(*s, dtype=dt, device="cuda").normal_(0.0, std, generator=g)
    x, wg, wu, wd = draw(1.0, R, H), draw(0.05, n, I, H), draw(0.05, n, I, H), draw(0.05, n, H, I)
    ends = np.cumsum([0] + list(counts))
    offsets = torch.tensor(ends, dtype=torch.int32, device="cuda")
    ws = torch.empty(moe.moe_workspace_bytes(cfg, R), dtype=torch.uint8, device="cuda")
    ys = [torch.full((R, H), float("nan"), dtype=dt, device="cuda") for _ in range(2)]
    for y in ys:
        moe.moe_expert_ffn(cfg, n, x, offsets, R, wg, wu, wd, None, None, None, y, ws)
    assert torch.equal(ys[0].view(bits), ys[1].view(bits))
    ref = torch.empty(R, H, dtype=torch.float64, device="cuda")
    for e in range(n):
        lo, hi = int(ends[e]), int(ends[e + 1])
        if lo == hi:
            continue
        xe = x[lo:hi].double()
        gate, up = (xe @ w[e].double().t().contiguous() for w in (wg, wu))
        h = gate * torch.sigmoid(gate) * up
        if act == "bf16":
            h = h.to(torch.bfloat16).double()
        ref[lo:hi] = h @ wd[e].double().t().contiguous()
    err = float((ys[0].double() - ref).abs().max() / ref.abs().max())
    print("experts", n, "rows", R, "H", H, "I", I, "err %.3e" % err, flush=True)
    # bf16: the output's rounding (2^-9), and intermediates that fall to the other side of a
    # rounding (2^-8 of one of I terms each); fp32: sums of at most H products, sqrt(H) * 2^-24 of
    # the largest value in the mean.  Both well inside the layer's bar.
    assert err <= TOL[act]


def _counts(n, lo, hi):
    c = np.random.default_rng(n * 1000 + hi).integers(lo, hi + 1, n)
    c[n // 3] = 0
    return c.tolist()


# Sizes that are no multiple of 64, by the kernel that the rules pick: weight streaming in
# both GEMMs past two rows per expert (270 tall tiles, a second round of CUs nearly empty) and at
# one or two; 128 x 512 tiles of GEMM-2 with a K and an N remainder: K up to 48, up to 384
# from three rows per expert, from 13 on, and 260 tiles of 53 K steps, four of them cut along K;
# 160- and 128-row tall tiles of long groups.
@pytest.mark.parametrize("counts,H,I", [
    (_counts(90, 0, 33), 520, 328), (_counts(90, 1, 5), 520, 328), (_counts(130, 1, 2), 136, 520),
    (_counts(128, 0, 9), 1000, 40), (_counts(128, 1, 20), 2056, 136), (_counts(128, 1, 70), 2056, 200),
    (_counts(52, 20, 60), 2504, 3400),
    ([900, 0, 513, 700], 328, 136), ([1500], 584, 264), ([300, 128, 129], 1032, 200)],
    ids=lambda v: str(v) if isinstance(v, int) else "%dx%d" % (len(v), sum(v)))
def test_bf16_ragged_rules(counts, H, I):
    _ffn(counts, H, I)


# K = 128 on either side of the launches that the short-K kernel takes: 2048 blocks (past twelve
# rows per expert) and 1024 (up to there); K = 64 with column blocks that are not halved further.
@pytest.mark.parametrize("counts,H,I", [
    (_counts(128, 1, 40), 2048, 128), (_counts(128, 1, 40), 1024, 128), ([144] * 8, 7168, 128),
    (_counts(128, 0, 7), 2048, 128), (_counts(64, 1, 1), 2048, 128), ([144] * 8, 7168, 64)],
    ids=lambda v: str(v) if isinstance(v, int) else "%dx%d" % (len(v), sum(v)))
def test_bf16_k128_rules(counts, H, I):
    _ffn(counts, H, I)


# fp32 past one tile per CU: one ring stage per workgroup for K of one, three and five chunks, the
# last one partly filled; and K up to 64 on the 64 x 64 tiles, GEMM-1 (1900 tiles) and GEMM-2
# (6400), with row, column and K remainders.
@pytest.mark.parametrize("counts,H,I", [
    (_counts(9, 60, 200), 520, 328), (_counts(30, 1, 90), 72, 264), (_counts(36, 400, 1300), 56, 40),
    (_counts(64, 1, 130), 1000, 24)],
    ids=lambda v: str(v) if isinstance(v, int) else "%dx%d" % (len(v), sum(v)))
def test_fp32_many_tiles(counts, H, I):
    _ffn(counts, H, I, "f32")


# The tile table's scan: expert counts on both sides of a wavefront's last expert and of the
# workgroup's, the first and last experts empty, up to one tile each but for one of several.
@pytest.mark.parametrize("act", ["f32", "bf16"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 129, 449, 512])
def test_tile_of_expert(n, act):
    c = np.random.default_rng(n).integers(0, 3, n) * np.random.default_rng(n + 1).integers(1, 33, n)
    c[n // 2] = 400
    if n > 2:
        c[0] = c[-1] = 0
    _ffn(c.tolist(), 64, 72 if act == "f32" else 64, act)


# Tables in which a thread per tile looks its expert up (more than four tiles of an expert), the
# last expert with rows of its own on both sides of a wavefront's last expert.
@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 192, 512])
def test_tile_look_up_last_expert(n):
    c = np.random.default_rng(n).integers(0, 3, n)
    c[0], c[-1] = 170, 333
    _ffn(c.tolist(), 64, 72, "f32")


# e4m3 weights, 13 to 64 rows per expert on average: short tiles of one and two 32-row blocks, up to
# four tiles an expert, one to seven K blocks (fewer than a ring has stages, as many, more), column
# tiles of GEMM-2 half empty; and, in the last case, GEMM-1 on tall tiles cut along K.
@pytest.mark.parametrize("counts,H,I", [
    ([1, 31, 32, 33, 0, 64, 65, 30], 128, 256), ([96, 97, 128, 129, 0, 5, 20, 2], 384, 384),
    ([16, 200, 0, 1], 640, 896), ([40, 70, 0, 100], 3328, 128)])
def test_e4m3_short_tiles(counts, H, I):
    assert 12 < sum(counts) // len(counts) <= 64
    check_ffn(counts, H, I, TOL["fp8"], weight_dtype="fp8")
