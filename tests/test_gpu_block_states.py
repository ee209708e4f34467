"""fp32 tensors: H_i, Z_i from the states of all key blocks, as a product of the selection's complement (short heads, long
lists) or the totals less a gather, on both sides of the lines between the two and one block more or less than whole tiles; and
the states formed in the selection's launch or in one of their own, on both sides of that line."""
import pytest

from paper_2602_12675_amd import workloads as W
from test_gpu_backward import test_backward_matches_oracle as check_backward
from test_gpu_forward_f32 import test_forward_f32_matches_oracle as check_forward

pytestmark = pytest.mark.gpu

BASE = W.TINY.replace(H=1, per_head_freq=True)
CASES = [
    BASE.replace(name="d64-64-of-1", grid=(16, 16, 16), topk_frac=0.016),                                # T_n = 64, k = 1
    BASE.replace(name="d64-65-of-0", grid=(16, 16, 16), extra_tokens=1, topk_frac=0.0),                  # totals alone
    BASE.replace(name="d64-65-of-1", grid=(16, 16, 16), extra_tokens=1, topk_frac=0.016, block_q=128),   # gather; T_m = 33
    BASE.replace(name="d64-90-of-3", grid=(15, 16, 24), topk_frac=0.0334),                               # T_n = 30 k
    BASE.replace(name="d64-91-of-3", grid=(15, 16, 24), extra_tokens=33, topk_frac=0.0334, H=2),
    BASE.replace(name="d128-65-of-1", grid=(16, 16, 16), extra_tokens=31, topk_frac=0.016, d=128, block_q=128),
    BASE.replace(name="d128-31-of-4", grid=(8, 15, 16), extra_tokens=32, topk_frac=0.13, d=128),         # T_m = 31
    BASE.replace(name="d64-237-of-12-one-launch", grid=(16, 12, 79), topk_frac=0.05),                    # 15 + 4 + 237 workgroups
    BASE.replace(name="d64-238-of-12", grid=(16, 12, 79), extra_tokens=1, topk_frac=0.05),
    BASE.replace(name="d128-33-of-5", grid=(8, 16, 16), extra_tokens=33, topk_frac=0.15, d=128, H=3),    # T_m = 33
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_forward(w):
    check_forward(w)


@pytest.mark.parametrize("w", [CASES[2], CASES[5], CASES[9]], ids=lambda w: w.name)
def test_backward(w):
    check_backward(w, True, True)
