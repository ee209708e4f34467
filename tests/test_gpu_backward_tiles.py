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


# Key blocks in several groups of heads (over 48 MB of gathered rows each, the last one at least four rounds of places), lists far
# longer than the mean among them: workload, groups, heads a group, heads to compare.  tests/test_work_order.py holds the numbers
# against the rule.
GROUPS = W.TINY.replace(B=1, grid=(21, 30, 52), d=128, block_q=128, dtype="bf16", topk_frac=0.03)
GROUPED = [
    (GROUPS.replace(name="bf16-d128-one-group", H=3), 1, 2, (0, 1, 2)),
    (GROUPS.replace(name="bf16-d128-two-groups", H=7), 2, 2, (0, 2, 6)),                                    # 512 key blocks
    (GROUPS.replace(name="bf16-d128-three-groups", H=9, grid=(21, 30, 51), extra_tokens=540), 3, 2, (0, 3, 8)),   # 511: a short last run
    (GROUPS.replace(name="bf16-d128-six-groups", H=9, extra_tokens=65), 6, 1, (0, 4, 8)),                   # 513, one head a group
    (GROUPS.replace(name="bf16-d128-many-heads", H=64, grid=(1, 50, 80), topk_frac=0.05), 3, 16, (0, 17, 63)),    # 63 key blocks
]


def groups_match(w, heads):
    import torch
    from paper_2602_12675_amd import api
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v, go = (torch.randn((1, w.H, w.N, w.d), generator=gen, device="cuda") for _ in range(4))
    k[:, :, : w.N // 10] *= 3.0                      # a few key blocks that most query blocks select
    k[:, :, : w.N // 10] += q.mean(2, keepdim=True) * 40
    q, k, v, go = (x.bfloat16() for x in (q, k, v, go))
    rw = torch.randn((2, w.d, w.d), generator=gen, device="cuda") / w.d ** 0.5
    al = torch.rand((w.H,), generator=gen, device="cuda")

    def grads(h0, h1):
        p = api.make_params(1, h1 - h0, w.N, w.d, w.block_q, w.block_kv, w.topk_frac, dtype=api.SLA2_BF16,
                            flags=api.SLA2_FLAG_SAVE_FOR_BACKWARD)
        a = [x[:, h0:h1].contiguous() for x in (q, k, v)]
        out, ws, da = torch.empty_like(a[0]), api.alloc_workspace(p), torch.empty((h1 - h0,), device="cuda")
        d = [torch.full_like(x, float("nan")) for x in a]
        idx = torch.empty((1, h1 - h0, w.T_m, w.k), dtype=torch.int32, device="cuda")
        api.sla2_forward(p, *a, rw, al[h0:h1].contiguous(), out, block_idx=idx, workspace=ws)
        api.sla2_backward(p, *a, al[h0:h1].contiguous(), go[:, h0:h1].contiguous(), *d, da, ws)
        torch.cuda.synchronize()
        return d, idx

    whole, idx = grads(0, w.H)
    lengths = torch.stack([x.flatten().bincount(minlength=-(-w.N // 64)) for x in idx[0]])
    assert (lengths > max(3 * w.T_m * w.k / lengths.shape[1], w.T_m * w.k * w.H / 3072)).any()      # long lists, as work_order.h has it
    assert all(x.isfinite().all() for x in whole)
    for h in heads:
        for name, x, y in zip(("dq", "dk", "dv"), whole, grads(h, h + 1)[0]):
            x, y = x[:, h : h + 1].double(), y.double()
            assert (x - y).norm() <= 2.0 ** -7 * y.norm(), (name, h, ((x - y).norm() / y.norm()).item())


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_backward_at_tile_edges(w):
    check(w, True, True)


@pytest.mark.parametrize("w,some", [(x[0], x[3]) for x in GROUPED if x[0].H <= 8], ids=lambda x: getattr(x, "name", ""))
def test_backward_over_groups_of_heads(w, some):
    """Heads are independent: a call over several order groups gives what calls over single heads give.

    Not bit for bit: the forward pass splits the key/value totals by the number of heads, so that H_i, kept in bf16, may
    round to its neighbour (2^-8 of its value, which the linear products pass on), and so may the result (2^-8 again):
    2^-7 in the 2-norm of a head.  A key block left out or taken twice leaves whole blocks of 64 rows undefined; the
    results start as NaN."""
    groups_match(w, some)


@pytest.mark.parametrize("w,some", [(x[0], x[3]) for x in GROUPED if x[0].H > 8], ids=lambda x: getattr(x, "name", ""))
def test_backward_over_groups_and_xcds(w, some):
    """More heads than XCDs, whose runs of key blocks go round them: groups of one, two and sixteen heads."""
    groups_match(w, some)
