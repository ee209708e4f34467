"""d = 64 with 64-row blocks and FP8 scores: the attention kernel has two main loops, chosen by k T_n (2,500 is the last
product on the pipelined one).  Both sides of that line against the oracle, with a full and a ragged last key block, and
the shortest list that reaches the line."""
import numpy as np
import pytest

import sla2_oracle as O
from helpers import check_mask, rel_l2, rows_ok, run_forward
from paper_2602_12675_amd import workloads as W

pytestmark = pytest.mark.gpu

LINE = 2500
LOWBIT_REL_L2 = 5e-2                     # the low-bit tolerance of the forward tests
BASE = W.TINY.replace(dtype="bf16", d=64, block_q=64, H=1, per_head_freq=True)


@pytest.mark.parametrize("quant", ["fp8", "fp8v"])
@pytest.mark.parametrize("n,k", [(6400, 25), (6400, 26), (6337, 26), (65536, 2), (65473, 3)])
def test_both_loops_match_the_oracle(n, k, quant):
    import torch
    from paper_2602_12675_amd import api
    t_n = -(-n // 64)
    w = BASE.replace(name="loops-%d-%d-%s" % (n, k, quant), grid=(1, 1, n), topk_frac=k / t_n, quant=quant)
    assert w.k == k and w.T_n == t_n
    inp = W.generate(w)
    r = run_forward(api, torch, inp)
    blocks = sorted({0, 1, w.T_m // 2, w.T_m - 2, w.T_m - 1})
    o = O.forward_head(inp.values("q", 0, 0), inp.values("k", 0, 0), inp.values("v", 0, 0), inp.router_w[0].astype(np.float64),
                       inp.router_w[1].astype(np.float64), inp.alpha[0], w.topk_frac, 64, 64,
                       quant={"fp8": O.QUANT_FP8, "fp8v": O.QUANT_FP8_V}[quant], q_blocks=blocks)
    assert check_mask(r["idx"][0, 0], o["R"], o["sel"]) == 0
    for i in blocks:
        rows = slice(64 * i, min(n, 64 * (i + 1)))
        assert rel_l2(r["out"][0, 0, rows], o["O"][rows]) <= LOWBIT_REL_L2
        rows_ok(r["out"][0, 0, rows], o["O"][rows], quant)
        np.testing.assert_allclose(r["lse"][0, 0, rows], o["L"][rows], rtol=0, atol=2e-2)
    assert not np.isnan(r["out"]).any()


def test_the_cases_lie_on_both_sides_of_the_line():
    assert [k * -(-n // 64) > LINE for n, k in ((6400, 25), (6400, 26), (6337, 26), (65536, 2), (65473, 3))] == [False, True, True, False, True]
