"""fp32 tensors, small calls at d = 64: H_i, Z_i and the totals formed by the attention kernel from the states of all key blocks, at the
ends of its range (1 and 16 key blocks, 17 beyond it), at remainders of four states, with no block and every block selected,
several query blocks or row groups a head; kept for the backward pass."""
import pytest

from paper_2602_12675_amd import workloads as W
from test_gpu_backward import test_backward_matches_oracle as check_backward
from test_gpu_forward_f32 import test_forward_f32_matches_oracle as check_forward

pytestmark = pytest.mark.gpu

BASE = W.TINY.replace(H=2, per_head_freq=True)
CASES = [
    BASE.replace(name="1-of-1", grid=(1, 1, 33), topk_frac=1.0),
    BASE.replace(name="1-of-2", grid=(1, 8, 8), extra_tokens=1, topk_frac=0.5, block_q=128),
    BASE.replace(name="0-of-5", grid=(5, 8, 8), topk_frac=0.0, H=3),
    BASE.replace(name="15-of-15", grid=(15, 8, 8), topk_frac=1.0),
    BASE.replace(name="2-of-16", grid=(16, 8, 8), topk_frac=0.1, B=2),
    BASE.replace(name="15-of-16-bq128", grid=(15, 8, 8), extra_tokens=33, topk_frac=0.95, block_q=128),      # T_m = 8, a part of the last
    BASE.replace(name="3-of-17", grid=(16, 8, 8), extra_tokens=1, topk_frac=0.2),                            # the product
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_forward(w):
    check_forward(w)


@pytest.mark.parametrize("w", [CASES[1], CASES[2], CASES[4], CASES[5]], ids=lambda w: w.name)
def test_backward(w):
    check_backward(w, True, True)
