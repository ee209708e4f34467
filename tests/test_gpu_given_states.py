"""Long lists at d = 128 with 128-row blocks: H_i formed before the attention kernel, as a product of the selection's complement
with the states of all key blocks in three bf16 parts - every mode, ragged ends, around whole tiles of 128 query blocks and 32 key
blocks, every block but one and every block selected, the training call, and more heads than one group holds."""
import numpy as np
import pytest

from paper_2602_12675_amd import workloads as W
from helpers import rel_l2
from test_gpu_backward import test_backward_matches_oracle as check_backward
from test_gpu_forward_bf16 import test_forward_bf16_matches_oracle as check_bf16
from test_gpu_forward_fp8 import test_forward_fp8_matches_oracle as check_fp8
from test_gpu_forward_fp8v import test_forward_fp8v_matches_oracle as check_fp8v
from test_gpu_forward_int8 import test_forward_int8_matches_oracle as check_int8

pytestmark = pytest.mark.gpu

BASE = W.TINY.replace(dtype="bf16", per_head_freq=True, d=128, block_q=128, H=1)
CASES = [   # k of T_n key blocks; the line is k > 40 + 0.025 T_n, 0.034 T_n in the low-bit modes
    (BASE.replace(name="44-of-64", grid=(16, 16, 16), topk_frac=0.69, H=2), check_bf16),                            # T_m = 32
    (BASE.replace(name="41-of-64-below", grid=(16, 16, 16), topk_frac=0.64), check_bf16),
    (BASE.replace(name="64-of-65", grid=(16, 16, 16), extra_tokens=1, topk_frac=0.985, B=2), check_bf16),           # T_m = 33
    (BASE.replace(name="63-of-63", grid=(63, 8, 8), topk_frac=1.0), check_bf16),
    (BASE.replace(name="60-of-257", grid=(64, 16, 16), extra_tokens=33, topk_frac=0.2335), check_bf16),             # T_m = 129
    (BASE.replace(name="fp8-60-of-97", grid=(24, 16, 16), extra_tokens=31, topk_frac=0.62, quant="fp8"), check_fp8),
    (BASE.replace(name="int8-60-of-97", grid=(24, 16, 16), extra_tokens=31, topk_frac=0.62, quant="int8"), check_int8),
    (BASE.replace(name="fp8v-60-of-97", grid=(24, 16, 16), extra_tokens=31, topk_frac=0.62, quant="fp8v"), check_fp8v),
]


@pytest.mark.parametrize("w,check", CASES, ids=lambda x: x.name if hasattr(x, "name") else "")
def test_forward(w, check):
    check(w)


@pytest.mark.parametrize("quant", ["none", "fp8"])
def test_backward(quant):
    check_backward(BASE.replace(name="train-45-of-66", grid=(16, 16, 16), extra_tokens=70, topk_frac=0.68, H=2, quant=quant), True, True)


def test_groups_of_heads():
    """160 heads of 64 key blocks: 6.3 MB of states each.  The call against two of 80 heads: only the order of the
    sums of Z_total differs (1e-7), which moves an output across a bf16 boundary now and then."""
    import torch
    from paper_2602_12675_amd import api
    H, N, d = 160, 4096, 128
    gen = torch.Generator(device="cuda").manual_seed(7)
    q, k, v = (torch.randn((1, H, N, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    rw = torch.randn((2, d, d), generator=gen, device="cuda") / d ** 0.5
    alpha = torch.rand((H,), generator=gen, device="cuda")

    def call(h0, h1):
        p = api.make_params(1, h1 - h0, N, d, 128, 64, 0.75, dtype=api.SLA2_BF16)
        out = torch.empty_like(q[:, h0:h1])
        api.sla2_forward(p, q[:, h0:h1], k[:, h0:h1], v[:, h0:h1], rw, alpha[h0:h1], out, workspace=api.alloc_workspace(p))
        return out.float().cpu().numpy()

    whole, parts = call(0, H), np.concatenate([call(0, H // 2), call(H // 2, H)], axis=1)
    for h in range(H):
        assert rel_l2(whole[0, h], parts[0, h]) < 2e-4, h


@pytest.mark.parametrize("H,frac", [(48, 1.0), (2, 0.1)])
def test_kphi_in_the_workspace(H, frac):
    """sla2_ws_layout.k_phi holds K^phi as fragments or has no bytes, whatever the lists' length (here the longest and a short one)."""
    import torch
    from paper_2602_12675_amd import api
    N, d, T_n = 4096, 128, 64
    gen = torch.Generator(device="cuda").manual_seed(7)
    q, k, v = (torch.randn((1, H, N, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    p = api.make_params(1, H, N, d, 128, 64, frac, dtype=api.SLA2_BF16)
    ws, L = api.alloc_workspace(p), api.sla2_workspace_layout(p)
    api.sla2_forward(p, q, k, v, torch.eye(d, device="cuda").repeat(2, 1, 1), torch.ones((H,), device="cuda"), torch.empty_like(q), workspace=ws)
    if L.z_blocks == L.k_phi:
        return
    got = api.workspace_view(ws, L.k_phi, torch.bfloat16, (H, T_n, d // 32, 4, 2, 32, 2, 4)).float().cpu().numpy()   # mt, ks, l / 32, l % 32, i / 4, i % 4
    got = got.transpose(0, 1, 3, 6, 4, 7, 2, 5).reshape(H, N, d)                # tokens 16 ks + 8 (i / 4) + 4 (l / 32) + i % 4
    kd = k[0].double()
    want = torch.softmax(kd - kd.mean(dim=1, keepdim=True), dim=-1).cpu().numpy()
    assert rel_l2(got, want) < 4e-3                                              # rounded to bf16: at most 2^-9 each
