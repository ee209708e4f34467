"""Sums of the linear branch over the blocks that are not selected, formed as a product of a bit matrix with all states:
one row, column group and 64-block step more or less than whole ones, no block and every block selected."""
import pytest

from paper_2602_12675_amd import workloads as W
from test_gpu_backward import test_backward_matches_oracle as check

pytestmark = pytest.mark.gpu

BASE = W.TINY.replace(per_head_freq=True, H=1, dtype="bf16")
CASES = [
    BASE.replace(name="d64-bq128-64-by-128", grid=(32, 16, 16), block_q=128, topk_frac=0.05),                        # T_m = 64, T_n = 128
    BASE.replace(name="d64-bq128-65-by-129", grid=(32, 16, 16), extra_tokens=1, block_q=128, topk_frac=0.3),         # T_m = 65, T_n = 129
    BASE.replace(name="d64-bq64-63-by-63", grid=(63, 8, 8), topk_frac=0.1),
    BASE.replace(name="d128-bq64-33-by-33", grid=(32, 8, 8), extra_tokens=7, d=128, topk_frac=0.2),
    BASE.replace(name="d128-bq128-1-by-2", grid=(1, 8, 16), d=128, block_q=128, topk_frac=0.5),
    BASE.replace(name="d128-none", grid=(3, 8, 8), d=128, topk_frac=0.0),
    BASE.replace(name="d64-every", grid=(3, 8, 8), topk_frac=1.0),
    BASE.replace(name="d64-two-heads", H=2, B=2, grid=(4, 8, 8), extra_tokens=3, topk_frac=0.4),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_backward_sums(w):
    check(w, True, True)
