"""Backward pass at the edges of its kernels' tiles: query blocks whose second 64-row half is empty, one-token last key
blocks, more query blocks than one 32-bit word of a column holds, every tile shape of the fp32 kernels."""
import pytest

from paper_2602_12675_amd import workloads as W
from test_gpu_backward import test_backward_matches_oracle as check

pytestmark = pytest.mark.gpu

BASE = W.TINY.replace(per_head_freq=True, H=1)
CASES = [
    BASE.replace(name="f32-d64-bq128-one-row", grid=(1, 8, 16), extra_tokens=1, block_q=128, topk_frac=0.4),       # N = 129
    BASE.replace(name="f32-d128-bq64-one-row", grid=(1, 8, 8), extra_tokens=1, d=128, topk_frac=0.5),              # N = 65
    BASE.replace(name="f32-d128-bq128-half-block", grid=(5, 8, 8), d=128, block_q=128, topk_frac=0.4),             # N = 320
    BASE.replace(name="f32-d64-37-blocks", grid=(36, 8, 8), extra_tokens=5, topk_frac=0.06),                       # N = 2309
    BASE.replace(name="bf16-d128-bq128-one-row", grid=(1, 16, 16), extra_tokens=1, d=128, block_q=128, dtype="bf16", topk_frac=0.4),
    BASE.replace(name="bf16-d64-bq64-35-blocks", grid=(34, 8, 8), extra_tokens=1, dtype="bf16", topk_frac=0.95),   # N = 2177, long lists
    BASE.replace(name="bf16-d128-bq64-33-blocks", grid=(33, 8, 8), d=128, dtype="bf16", topk_frac=0.1),            # N = 2112
    BASE.replace(name="bf16-d64-bq128-half-block", grid=(5, 8, 8), block_q=128, dtype="bf16", topk_frac=0.4),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_backward_at_tile_edges(w):
    check(w, True, True)
