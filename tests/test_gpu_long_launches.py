"""Launches of 2^32 threads and more, which a one-dimensional grid does not take: small rows of
very many tokens, checked on both ends and in the middle."""
import pytest
import torch

import paper_2601_08800_amd as moe

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _give_memory_back():
    torch.cuda.empty_cache()
    yield
    torch.cuda.empty_cache()


def _cfg(H, E, k, I, act):
    return moe.MoEConfig(hidden=H, n_experts=E, top_k=k, score_fn=moe.MOE_SCORE_SOFTMAX, renormalize=1, routed_scale=1.0,
                         n_groups=1, topk_groups=1, group_score_n=0, expert_lo=0, expert_hi=E, inter_local=I,
                         act_dtype=act, weight_dtype=act)


def _sample(n):
    return torch.cat([torch.arange(0, 300), torch.arange(n // 2, n // 2 + 300), torch.arange(n - 300, n)]).cuda()


def test_combine_of_2_to_the_26_row_segments():
    T, H, rows = (1 << 25) + 3, 520, 1000                 # two wavefronts a row; 70 GB of output
    g = torch.Generator(device="cuda").manual_seed(1)
    ys = torch.empty(rows, H, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    inv = torch.randint(-1, rows, (T, 1), dtype=torch.int32, device="cuda", generator=g)
    w = torch.rand(T, 1, device="cuda", generator=g)
    out = torch.empty(T, H, device="cuda")
    at = _sample(T)
    out[at] = float("nan")
    moe.moe_combine(_cfg(H, 8, 1, 128, moe.MOE_BF16), T, ys, inv, w, None, out)
    pos = inv[at, 0].long()
    assert torch.equal(out[at], torch.where(pos[:, None] >= 0, ys[pos.clamp(min=0)].float() * w[at], 0.0))


def test_exact_gate_of_2_to_the_22_tiles():
    T, E, H, k = (1 << 21) + 5, 512, 8, 4                 # 8.6 GB of logits
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.empty(T, H, device="cuda").normal_(generator=g)
    gate_w = torch.empty(E, H, device="cuda").normal_(generator=g)
    cfg = _cfg(H, E, k, 128, moe.MOE_F32)
    ids = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.empty(T, k, device="cuda")
    ws = torch.empty(moe.moe_workspace_bytes(cfg, T), dtype=torch.uint8, device="cuda")
    moe.moe_route(cfg, T, x, gate_w, None, None, None, ids, w, ws)
    at = _sample(T)
    top = (x[at].double() @ gate_w.double().t().contiguous()).topk(k, dim=1)
    assert torch.equal(ids[at].long(), top.indices)
    want = torch.softmax(top.values, dim=1)
    assert float(((w[at].double() - want).abs() / want).max()) <= 2.0 ** -24 + 2.0 ** -35


def test_fp32_ffn_of_2_to_the_24_tiles():
    R, H, I = 1 << 20, 72, 16384                          # 64 GB of intermediate in the workspace
    g = torch.Generator(device="cuda").manual_seed(3)
    draw = lambda std, *s: torch.empty(*s, device="cuda").normal_(0.0, std, generator=g)
    x, wg, wu, wd = draw(1.0, R, H), draw(0.1, 1, I, H), draw(0.1, 1, I, H), draw(0.1, 1, H, I)
    cfg = _cfg(H, 1, 1, I, moe.MOE_F32)
    offsets = torch.tensor([0, R], dtype=torch.int32, device="cuda")
    ys = torch.full((R, H), float("nan"), device="cuda")
    ws = torch.empty(moe.moe_workspace_bytes(cfg, R), dtype=torch.uint8, device="cuda")
    moe.moe_expert_ffn(cfg, 1, x, offsets, R, wg, wu, wd, None, None, None, ys, ws)
    assert not torch.isnan(ys).any()
    at = _sample(R)
    gate, up = (x[at].double() @ m[0].double().t().contiguous() for m in (wg, wu))
    ref = (gate * torch.sigmoid(gate) * up) @ wd[0].double().t().contiguous()
    assert float((ys[at].double() - ref).abs().max() / ref.abs().max()) <= 1e-5
