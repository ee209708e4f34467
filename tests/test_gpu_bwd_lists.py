"""The lists of the key side, made by the first workgroups of the query side's launch: 64 columns of a head by one workgroup of
128 or 256 threads, filled up to whole rounds of eight.  One column, word and head more or less than whole ones."""
import pytest

from paper_2602_12675_amd import workloads as W
from test_gpu_backward import test_backward_matches_oracle as check

pytestmark = pytest.mark.gpu

BASE = W.TINY.replace(per_head_freq=True, H=1)
CASES = [
    BASE.replace(name="f32-d64-64-by-64", grid=(64, 8, 8), topk_frac=0.1),                                              # one job
    BASE.replace(name="f32-d64-65-by-65", grid=(64, 8, 8), extra_tokens=1, topk_frac=0.1, H=4),                         # eight jobs
    BASE.replace(name="f32-d128-33-by-65", grid=(64, 8, 8), extra_tokens=9, d=128, block_q=128, topk_frac=0.3, H=5),    # ten
    BASE.replace(name="bf16-d64-bq64-65-by-65", grid=(64, 8, 8), extra_tokens=1, topk_frac=0.1, H=3, dtype="bf16"),     # 128 threads
    BASE.replace(name="bf16-d128-bq64-32-by-32", grid=(32, 8, 8), d=128, topk_frac=1.0, H=9, dtype="bf16"),             # nine, every block
    # one query block (of one token, dQ is zero in exact arithmetic and 1e-12 here: a relative bound holds from two tokens on)
    BASE.replace(name="bf16-d64-bq128-1-by-2", grid=(1, 8, 16), block_q=128, topk_frac=0.5, dtype="bf16"),
    BASE.replace(name="f32-d64-none", grid=(3, 8, 8), topk_frac=0.0),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_lists_with_the_query_side(w):
    check(w, True, True)
