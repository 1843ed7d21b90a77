"""Index kernels at the edges of their tiles: the two launches of the dispatch index
around their chunk of 1024 assignments, and the combine's batches of eight rows."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_dispatch, dev, make_layer
from workloads import gen

pytestmark = pytest.mark.gpu

NO_WEIGHTS = {"w_gate": None, "w_up": None, "w_down": None}


# one run, whole and ragged runs, more than 256 runs (chunks of two); one local expert,
# 512 of them, an expert count that does not divide the workgroup
@pytest.mark.parametrize("T,k,E,lo,hi", [
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
