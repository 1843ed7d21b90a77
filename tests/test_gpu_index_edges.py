"""Routing and index kernels at the edges of their tiles and of the rules that pick
them: the exact gate's 16 x 16 tiles and K groups, the two launches of the dispatch
index around their chunk of 1024 assignments, and the combine's batches of eight rows."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_dispatch, check_routing, dev, host, make_layer, oracle_route
from workloads import gen

pytestmark = pytest.mark.gpu

NO_WEIGHTS = {"w_gate": None, "w_up": None, "w_down": None}


# The exact gate in its three forms (one launch: up to 256 tokens and 64 experts; rows: few tokens
# or long gate rows; tiles: the rest).  Tokens and experts one below, at and one above a tile; rows
# of one piece, of a partial group of pieces, of a second round of 256 and 512 pieces, and of more
# groups than a workgroup has wavefronts; grouped gates in every form.
@pytest.mark.parametrize("act,T,E,H,k,G", [
    ("bf16", 1, 1, 8, 1, 1), ("bf16", 15, 17, 40, 3, 1), ("bf16", 16, 16, 264, 16, 1),
    ("bf16", 17, 33, 2056, 5, 1), ("bf16", 333, 128, 520, 8, 1), ("bf16", 500, 512, 72, 32, 1),
    ("bf16", 49, 64, 1024, 6, 8), ("bf16", 50, 48, 136, 5, 4), ("bf16", 21, 256, 4104, 8, 8),
    ("bf16", 256, 8, 1032, 2, 1), ("bf16", 257, 8, 1032, 2, 1), ("bf16", 200, 64, 2056, 6, 8),
    ("bf16", 140, 64, 2048, 6, 1), ("bf16", 3, 128, 7176, 8, 1), ("bf16", 2, 130, 4104, 6, 1),
    ("f32", 256, 8, 264, 2, 1), ("f32", 257, 8, 264, 2, 1), ("f32", 31, 130, 1032, 8, 1),
    ("f32", 5000, 16, 8, 3, 1), ("f32", 65, 96, 2048, 4, 6), ("f32", 7, 61, 2056, 4, 1),
    ("f32", 130, 64, 1024, 4, 8), ("f32", 400, 3, 2056, 1, 1)])
def test_exact_route_tiles(act, T, E, H, k, G):
    base = gen.CONFIGS["c4" if G > 1 else "c1"]
    w = base.replace(name="exact_tiles", T=T, E=E, H=H, k=k, I=8, act_dtype=act, weight_dtype=act, tp=1,
                     expert_lo=0, expert_hi=E, shared_expert=False, n_groups=G,
                     topk_groups=max(1, G // 2), group_score_n=2 if G > 1 else 0, seed=T + E)
    x, gate = gen.make_x(w), gen.make_gate(w)
    L = make_layer(w, {"gate": gate, "experts": NO_WEIGHTS, "shared": None})
    L.route(dev(x))
    torch.cuda.synchronize()
    assert int(L.ws[:4].view(torch.int32).item()) == 0          # exact keys: nothing to re-score
    ids_ref, w_ref, margin = oracle_route(w, x, gate)
    check_routing(host(L.topk_ids), host(L.topk_w), ids_ref, w_ref, margin, w.routed_scale, "exact_tiles")


# one run, whole and ragged runs, more than 256 runs (chunks of two); one local expert,
# 512 of them, an expert count that does not divide the workgroup; top-1 on either side of the
# 2048 tokens of the one-launch form
@pytest.mark.parametrize("T,k,E,lo,hi", [
    (2048, 1, 40, 0, 40), (2049, 1, 40, 3, 40), (4096, 1, 8, 0, 8),
    (4097, 1, 512, 0, 512), (4097, 1, 512, 511, 512), (2560, 2, 300, 0, 300), (1366, 3, 96, 5, 42),
    (33000, 8, 64, 0, 64), (262145, 1, 32, 3, 32), (32768, 8, 8, 0, 8)])
def test_dispatch_index_runs(T, k, E, lo, hi):
    w = gen.CONFIGS["c2d"].replace(T=T, H=8, E=E, k=k, I=8, expert_lo=lo, expert_hi=hi)
    rng = np.random.default_rng(T + E)
    ids = rng.random((T, E), dtype=np.float32).argpartition(k - 1, axis=1)[:, :k].astype(np.int32)
    ids[: T // 3, 0] = lo                                    # a hot expert (a token may hold it twice)
    d = {"x": gen.make_x(w), "gate": gen.make_gate(w), "experts": NO_WEIGHTS, "shared": None}
    L = make_layer(w, d)
    L.topk_ids = dev(ids)
    L.dispatch(dev(d["x"]))
    torch.cuda.synchronize()
    check_dispatch(L, ids, w, d["x"])


# rows of one piece, of one wavefront's 64 pieces and one more; 1, 8, 9 and 32 experts a
# token.  fp32 sums of at most 33 products of bf16 values: 33 * 2^-24 of the sum of magnitudes.
@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("H,k", [(8, 1), (512, 8), (520, 9), (1032, 32)])
def test_combine_row_batches(H, k, shared):
    T, E = 37, 40
    w = gen.CONFIGS["c2d"].replace(T=T, H=H, E=E, k=k, I=8, expert_lo=0, expert_hi=33)
    rng = np.random.default_rng(H + k)
    ids = np.stack([rng.permutation(E)[:k] for _ in range(T)]).astype(np.int32)
    L = make_layer(w, {"gate": gen.make_gate(w), "experts": NO_WEIGHTS, "shared": None})
    _, _, _, inv, _ = oracle.dispatch(ids, None, 0, 33, want_xs=False)
    tw = rng.random((T, k), dtype=np.float32)
    g = torch.Generator(device="cuda").manual_seed(H)
    L.ys.normal_(generator=g)
    L.inv, L.topk_w = dev(inv.reshape(-1).astype(np.int32)), dev(tw)
    ref = torch.zeros(T, H, dtype=torch.float64, device="cuda")
    mag = torch.zeros_like(ref)
    if shared:
        L.shared_ys = torch.empty(T, H, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
        ref += L.shared_ys.double()
        mag += L.shared_ys.double().abs()
    for j in range(k):
        pos = L.inv.view(T, k)[:, j].long()
        term = L.ys[pos.clamp(min=0)].double() * (L.topk_w[:, j].double() * (pos >= 0))[:, None]
        ref += term
        mag += term.abs()
    L.out.fill_(float("nan"))
    L.combine()
    assert bool(((L.out.double() - ref).abs() <= 33 * 2.0 ** -24 * mag).all())
