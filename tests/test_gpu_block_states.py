"""fp32 tensors: H_i, Z_i from the states of all key blocks, as a product of the selection's complement (short heads, long
lists) or the totals less a gather, on both sides of the lines between the two and one block more or less than whole tiles; and
the states formed in the selection's launch or in one of their own, on both sides of that line."""
import numpy as np
import pytest

import sla2_oracle as O
from paper_2602_12675_amd import workloads as W
from helpers import rel_l2
from test_gpu_backward import test_backward_matches_oracle as check_backward
from test_gpu_forward_f32 import test_forward_f32_matches_oracle as check_forward

pytestmark = pytest.mark.gpu

BASE = W.TINY.replace(H=1, per_head_freq=True)
CASES = [
    BASE.replace(name="d64-64-of-1", grid=(16, 16, 16), topk_frac=0.016),                                # T_n = 64, k = 1
    BASE.replace(name="d64-65-of-0", grid=(16, 16, 16), extra_tokens=1, topk_frac=0.0),                  # totals alone
    BASE.replace(name="d64-65-of-1", grid=(16, 16, 16), extra_tokens=1, topk_frac=0.016, block_q=128),   # gather; T_m = 33
    BASE.replace(name="d64-90-of-3", grid=(15, 16, 24), topk_frac=0.0334),                               # gather
    BASE.replace(name="d64-91-of-3", grid=(15, 16, 24), extra_tokens=33, topk_frac=0.0334, H=2),
    BASE.replace(name="d128-65-of-1", grid=(16, 16, 16), extra_tokens=31, topk_frac=0.016, d=128, block_q=128),
    BASE.replace(name="d128-31-of-4", grid=(8, 15, 16), extra_tokens=32, topk_frac=0.13, d=128),         # T_m = 31
    BASE.replace(name="d64-237-of-12-one-launch", grid=(16, 12, 79), topk_frac=0.05),                    # 15 + 4 + 237 workgroups
    BASE.replace(name="d64-238-of-12", grid=(16, 12, 79), extra_tokens=1, topk_frac=0.05),
    BASE.replace(name="d64-80-of-5", grid=(20, 16, 16), topk_frac=0.0625),                               # T_n = 16 k: the product
    BASE.replace(name="d64-81-of-5", grid=(20, 16, 16), extra_tokens=9, topk_frac=0.0617),               # gather
    BASE.replace(name="d128-75-of-3", grid=(15, 16, 20), topk_frac=0.04, d=128, block_q=128),            # T_n = 25 k: the product
    BASE.replace(name="d128-76-of-3", grid=(15, 16, 20), extra_tokens=33, topk_frac=0.0395, d=128, block_q=128),   # gather
    BASE.replace(name="d128-33-of-5", grid=(8, 16, 16), extra_tokens=33, topk_frac=0.15, d=128, H=3),    # T_m = 33
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_forward(w):
    check_forward(w)


@pytest.mark.parametrize("w", [CASES[2], CASES[5]] + CASES[9:], ids=lambda w: w.name)
def test_backward(w):
    check_backward(w, True, True)


@pytest.mark.parametrize("H,train", [(22, False), (31, True)])
def test_groups_of_heads(H, train):
    """Two batches of 22 heads of 64 key and 32 query blocks, 6.3 MB of states each: 40 heads and 4, the second batch in both groups;
    training, without H_i, 4.2 MB: 60 heads and 2."""
    import torch
    from paper_2602_12675_amd import api
    B, N, d, frac = 2, 4096, 128, 0.1
    gen = torch.Generator(device="cuda").manual_seed(13)
    q, k, v, dout = (torch.randn((B, H, N, d), generator=gen, device="cuda") for _ in range(4))
    rw, alpha = torch.randn((2, d, d), generator=gen, device="cuda") / d ** 0.5, torch.rand((H,), generator=gen, device="cuda")
    p = api.make_params(B, H, N, d, 128, 64, frac, dtype=api.SLA2_F32, flags=api.SLA2_FLAG_SAVE_FOR_BACKWARD if train else 0)
    ws, out = api.alloc_workspace(p), torch.empty_like(q)
    idx = torch.empty((B, H, N // 128, api.sla2_num_selected(p)), dtype=torch.int32, device="cuda")
    api.sla2_forward(p, q, k, v, rw, alpha, out, block_idx=idx, workspace=ws)
    if train:
        dq, dk, dv = (torch.empty_like(q) for _ in range(3))
        api.sla2_backward(p, q, k, v, alpha, dout, dq, dk, dv, torch.empty_like(alpha), ws)
    L = api.sla2_workspace_layout(p)
    totals = api.workspace_view(ws, L.h_total, torch.float32, (B, H, d, d))
    Wq, Wk = rw.double().cpu().numpy()
    for x in (0, 21, 39, 40, 43) if not train else (0, 59, 60, 61):
        b, h = divmod(x, H)
        Q, K, V, G = (t[b, h].double().cpu().numpy() for t in (q, k, v, dout))
        sel, some = idx[b, h].cpu().numpy(), [0, 15, 31]
        rows = np.concatenate([np.arange(128 * i, 128 * i + 128) for i in some])
        o = O.forward_head(Q, K, V, Wq, Wk, float(alpha[h]), frac, 128, 64, q_blocks=some, sel=sel)
        assert rel_l2(out[b, h].cpu().numpy()[rows], o["O"][rows]) < 2e-6, x
        h_j, _ = O.kv_state(O.phi(O.smooth_k(K)), V, 64)
        assert rel_l2(totals[b, h].cpu().numpy(), h_j.sum(axis=0)) < 2e-6, x
        if train:
            g = O.backward_head(Q, K, V, sel, float(alpha[h]), G, 128, 64)
            for name, t in (("dQ", dq), ("dK", dk), ("dV", dv)):
                assert rel_l2(t[b, h].cpu().numpy(), g[name]) < 3e-5, (x, name)
