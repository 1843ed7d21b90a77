"""Which arithmetic the router answers with, and at sizes where its launches are long."""
import numpy as np
import pytest
import torch

import paper_2601_08800_amd as moe

pytestmark = pytest.mark.gpu


def _cfg(T, E, H, k, act=moe.MOE_BF16, renorm=1, **kw):
    d = dict(hidden=H, n_experts=E, top_k=k, score_fn=moe.MOE_SCORE_SOFTMAX, renormalize=renorm, routed_scale=1.0,
             n_groups=1, topk_groups=1, group_score_n=0, expert_lo=0, expert_hi=E, inter_local=128, act_dtype=act,
             weight_dtype=act)
    d.update(kw)
    return moe.MoEConfig(**d)


def _route(cfg, T, x, gate_w, select_bias=None):
    ids = torch.empty(T, cfg.top_k, dtype=torch.int32, device="cuda")
    w = torch.empty(T, cfg.top_k, device="cuda")
    ws = torch.empty(moe.moe_workspace_bytes(cfg, T), dtype=torch.uint8, device="cuda")
    moe.moe_route(cfg, T, x, gate_w, None, select_bias, None, ids, w, ws)
    torch.cuda.synchronize()
    return ids, w, int(ws[:4].view(torch.int32).item())


# bf16 batches up to 4096 tokens whose logits are fp64: T*E*H up to 5 * 2^25, and up to 2^28 for
# gate rows past E*H = 2^19.  Among them more 16 x 16 tiles than 1024 (short rows), and token
# counts just past a multiple of 16 (long rows).  The weights are then those of fp64
# arithmetic, rounded once: 2^-24, and 2^-35 for the fp64 sums' own error (H * 2^-53 of the sum of
# magnitudes, below 2^-36 here).
@pytest.mark.parametrize("T,E,H,k", [(2304, 128, 512, 8), (1200, 256, 512, 8), (4096, 64, 640, 6),
                                     (4096, 512, 72, 8), (33, 512, 14336, 8), (511, 512, 1024, 4)])
@pytest.mark.parametrize("renorm", [0, 1])
def test_bf16_batches_with_fp64_weights(T, E, H, k, renorm):
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.empty(T, H, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    gate_w = torch.empty(E, H, dtype=torch.bfloat16, device="cuda").normal_(0.0, H ** -0.5, generator=g)
    ids, w, rescored = _route(_cfg(T, E, H, k, renorm=renorm), T, x, gate_w)
    assert rescored == 0
    z = x.double() @ gate_w.double().t().contiguous()
    top = z.topk(k, dim=1)
    assert torch.equal(ids.long(), top.indices)
    ref = torch.softmax(top.values if renorm else z, dim=1)
    if not renorm:
        ref = ref.gather(1, top.indices)
    err = float(((w.double() - ref).abs() / ref).max())
    print("T %d E %d H %d: largest relative error %.3g" % (T, E, H, err), flush=True)
    assert err <= 2.0 ** -24 + 2.0 ** -35


# The re-scoring list at its longest: gate rows in equal pairs, so that every token's picks
# tie and all tokens are listed, on both sides of the 512 that get a workgroup each; one to
# eight experts a lane, soft-max and sigmoid with a group limit.  Of a pair the lower expert comes first.
@pytest.mark.parametrize("T", [511, 512, 513, 770])
@pytest.mark.parametrize("E,H,G", [(64, 8264, 1), (64, 16392, 8), (128, 8200, 1), (256, 4104, 1), (256, 8200, 8),
                                   (512, 2056, 1), (512, 4104, 16)])
def test_every_token_is_rescored(E, H, G, T):
    g = torch.Generator(device="cuda").manual_seed(T + E)
    gs, k = E // G, 8
    x = torch.empty(T, H, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    half = torch.empty(G, gs // 2, H, dtype=torch.bfloat16, device="cuda").normal_(0.0, H ** -0.5, generator=g)
    gate_w = torch.cat([half, half], dim=1).reshape(E, H).contiguous()      # experts e and e + gs/2 of each group
    cfg = _cfg(T, E, H, k, **(dict(score_fn=moe.MOE_SCORE_SIGMOID, n_groups=G, topk_groups=G // 2, group_score_n=2)
                              if G > 1 else {}))
    ids, w, rescored = _route(cfg, T, x, gate_w)
    assert rescored == T
    z = x.double() @ half.reshape(E // 2, H).double().t().contiguous()
    key = torch.sigmoid(z) if G > 1 else z
    per = key.view(T, G, gs // 2)
    if G > 1:                                   # a group's two largest keys are a pair
        kept = per.max(dim=2).values.topk(G // 2, dim=1).indices
        per = per.masked_fill(~torch.zeros(T, G, dtype=torch.bool, device="cuda").scatter_(1, kept, True)[:, :, None],
                              float("-inf"))
    top = per.reshape(T, E // 2).topk(k // 2, dim=1)
    first = top.indices // (gs // 2) * gs + top.indices % (gs // 2)
    ref = torch.stack([first, first + gs // 2], dim=2).reshape(T, k)
    assert torch.equal(ids.long(), ref)
    sc = torch.gather(key, 1, top.indices).repeat_interleave(2, dim=1)
    want = torch.softmax(sc, dim=1) if G == 1 else sc / sc.sum(dim=1, keepdim=True)
    assert float(((w.double() - want).abs() / want).max()) <= 2.0 ** -24 + 2.0 ** -35
