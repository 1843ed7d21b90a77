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
