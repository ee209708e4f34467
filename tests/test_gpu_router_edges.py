"""GPU parity of the block selection, hard and soft, at the edges of its tiles: a ragged query block that is alone in its
tile of 16 or the last of a full one, a ragged key block at the ends of a 64-wide slot and of a round of 256, one, two and
three rounds (the score tiles take turns), numbers of workgroups that the eight XCDs do not divide.  The masks are the
oracle's outside its tie window; the soft masks agree to 1e-6, float32's rounding of a number below 1 times ten."""
import numpy as np
import pytest

import sla2_oracle as O
from helpers import check_mask
from paper_2602_12675_amd import workloads as W
from test_gpu_router import run_router
from test_gpu_router_soft import oracle_soft, run_soft

pytestmark = pytest.mark.gpu


def shape(blocks, last, d, H, block_q=64):               # `blocks` key blocks, the last of `last` tokens
    n = (blocks - 1) * 64 + last
    return W.TINY.replace(name=f"d{d}-{blocks}x64-last{last}-H{H}-bq{block_q}", grid=(1, 1, n), d=d, H=H, block_q=block_q,
                          topk_frac=0.2, dtype="bf16")


CASES = [shape(16, 64, 64, 1), shape(16, 1, 64, 3), shape(17, 33, 128, 3), shape(32, 63, 128, 5, 128), shape(33, 1, 128, 3, 128),
         shape(64, 1, 64, 3), shape(65, 1, 64, 2), shape(256, 7, 128, 1, 128), shape(257, 1, 128, 1, 128), shape(513, 9, 64, 1)]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_selection_at_the_edges(w):
    import torch
    from paper_2602_12675_amd import api
    inp = W.generate(w)
    _, _, idx, kk = run_router(api, torch, inp)
    soft, _ = run_soft(api, torch, inp, 0.1)
    Wq, Wk = inp.router_w[0].astype(np.float64), inp.router_w[1].astype(np.float64)
    for b in range(w.B):
        for h in range(w.H):
            R = O.router_scores(inp.values("q", b, h), O.smooth_k(inp.values("k", b, h)), Wq, Wk, w.block_q, w.block_kv)
            check_mask(idx[b, h], R, O.topk_rows(R, kk))
            np.testing.assert_allclose(soft[b, h], oracle_soft(inp, b, h, kk, 0.1), rtol=0, atol=1e-6)
