"""Long lists at d = 128 with 128-row blocks: H_i formed before the attention kernel, as a product of the selection's complement
with the states of all key blocks in three bf16 parts - every mode, ragged ends, around whole tiles of 128 query blocks and 32 key
blocks, every block but one and every block selected, the training call, and more heads than one group holds.  With one or two
heads (CASES, test_backward) the states are rebuilt in the attention kernel; MANY has enough heads for the product."""
import numpy as np
import pytest

import sla2_oracle as O
from paper_2602_12675_amd import workloads as W
from helpers import rel_l2, rows_ok
from test_gpu_backward import test_backward_matches_oracle as check_backward
from test_gpu_forward_bf16 import test_forward_bf16_matches_oracle as check_bf16
from test_gpu_forward_fp8 import test_forward_fp8_matches_oracle as check_fp8
from test_gpu_forward_fp8v import test_forward_fp8v_matches_oracle as check_fp8v
from test_gpu_forward_int8 import test_forward_int8_matches_oracle as check_int8

pytestmark = pytest.mark.gpu

BASE = W.TINY.replace(dtype="bf16", per_head_freq=True, d=128, block_q=128, H=1)
CASES = [   # k of T_n key blocks
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
    """160 heads below the line, 48 of 64 key blocks (groups of heads against the oracle: MANY).  The call against two of 80 heads: only
    the order of the sums of Z_total differs (1e-7), which moves an output across a bf16 boundary now and then."""
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


MANY = [   # H, N, k, mode
    (32, 6208, 66, "none"),                           # T_m = 49, T_n = 97
    (32, 6145, 96, "none"),                           # the last block of one token
    (32, 6208, 97, "none"),                           # every block
    (12, 16416, 80, "none"),                          # T_m = 129, T_n = 257
    (32, 6175, 72, "fp8"), (32, 6175, 72, "int8"), (32, 6175, 72, "fp8v"),
    (2, 131067, 400, "none"),                         # T_n = 2,048, the largest
    (84, 8192, 70, "none"),                           # 12.6 MB of states a head: 80 and 4 heads
]


def many(H, N, k, mode, flags=0):
    """The call on random heads; that it has no K^phi."""
    import torch
    from paper_2602_12675_amd import api
    d, T_n = 128, -(-N // 64)
    gen = torch.Generator(device="cuda").manual_seed(11)
    q, kk, v = (torch.randn((1, H, N, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    rw, alpha = torch.randn((2, d, d), generator=gen, device="cuda") / d ** 0.5, torch.rand((H,), generator=gen, device="cuda")
    p = api.make_params(1, H, N, d, 128, 64, k / T_n, dtype=api.SLA2_BF16, quant_mode=api.QUANT_MODES[mode], flags=flags)
    ws, L = api.alloc_workspace(p), api.sla2_workspace_layout(p)
    assert api.sla2_num_selected(p) == k and L.z_blocks == L.k_phi
    out, idx = torch.empty_like(q), torch.empty((1, H, -(-N // 128), k), dtype=torch.int32, device="cuda")
    api.sla2_forward(p, q, kk, v, rw, alpha, out, block_idx=idx, workspace=ws)
    return p, q, kk, v, rw, alpha, out, idx.cpu().numpy(), ws


@pytest.mark.parametrize("H,N,k,mode", MANY)
def test_forward_many_heads(H, N, k, mode):
    _, q, kk, v, rw, alpha, out, idx, _ = many(H, N, k, mode)
    quant = {"none": O.QUANT_NONE, "fp8": O.QUANT_FP8, "int8": O.QUANT_INT8, "fp8v": O.QUANT_FP8_V}[mode]
    T_m = idx.shape[2]
    some = [0, T_m // 2, T_m - 1]
    rows = np.concatenate([np.arange(128 * i, min(N, 128 * i + 128)) for i in some])
    Wq, Wk = rw.double().cpu().numpy()
    for h in {0, H - 1} if H < 84 else (0, 79, 80, 83):
        Q, K, V = (x[0, h].double().cpu().numpy() for x in (q, kk, v))
        ref = O.forward_head(Q, K, V, Wq, Wk, float(alpha[h]), k / -(-N // 64), 128, 64, quant=quant, q_blocks=some, sel=idx[0, h])["O"][rows]
        got = out[0, h].float().cpu().numpy()[rows]
        assert rel_l2(got, ref) <= (2e-2 if mode == "none" else 5e-2)   # those of the forward tests
        rows_ok(got, ref, mode)


@pytest.mark.parametrize("mode", ["none", "fp8"])
def test_backward_many_heads(mode):
    import torch
    from paper_2602_12675_amd import api
    H, N = 32, 6175
    p, q, kk, v, _, alpha, out, idx, ws = many(H, N, 75, mode, api.SLA2_FLAG_SAVE_FOR_BACKWARD)
    dout = torch.randn(q.shape, generator=torch.Generator(device="cuda").manual_seed(12), device="cuda").to(torch.bfloat16)
    dq, dk, dv = (torch.empty_like(q) for _ in range(3))
    dalpha = torch.empty_like(alpha)
    api.sla2_backward(p, q, kk, v, alpha, dout, dq, dk, dv, dalpha, ws)
    for h in (0, H - 1):
        g = O.backward_head(*(x[0, h].double().cpu().numpy() for x in (q, kk, v)), idx[0, h], float(alpha[h]),
                            dout[0, h].double().cpu().numpy(), 128, 64, quant=O.QUANT_FP8 if mode == "fp8" else O.QUANT_NONE)
        for name, got in (("dQ", dq), ("dK", dk), ("dV", dv)):
            assert rel_l2(got[0, h].float().cpu().numpy(), g[name]) < 2e-2, name


@pytest.mark.parametrize("H,T_n,frac", [(32, 97, 0.9), (2, 64, 0.1)])
def test_kphi_in_the_workspace(H, T_n, frac):
    """sla2_ws_layout.k_phi holds K^phi as fragments or has no bytes, whatever the lists' length (here a long one and a short one)."""
    import torch
    from paper_2602_12675_amd import api
    N, d = 64 * T_n, 128
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


@pytest.mark.parametrize("H,N,k,dtype", [(32, 6175, 75, "bfloat16"), (3, 2041, 5, "bfloat16"), (3, 2041, 5, "float32"), (2, 4999, 2, "float32")])
def test_second_backward_of_a_forward_call(H, N, k, dtype):
    """dH_j lies in the forward pass's scratch: a second backward call finds all that the forward call kept.  Long and short bf16
    lists, the fp32 product and gather."""
    import torch
    from paper_2602_12675_amd import api
    d = 128
    gen = torch.Generator(device="cuda").manual_seed(14)
    q, kk, v, dout = (torch.randn((1, H, N, d), generator=gen, device="cuda").to(getattr(torch, dtype)) for _ in range(4))
    rw, alpha = torch.randn((2, d, d), generator=gen, device="cuda") / d ** 0.5, torch.rand((H,), generator=gen, device="cuda")
    p = api.make_params(1, H, N, d, 128, 64, k / -(-N // 64), dtype=api.SLA2_BF16 if dtype == "bfloat16" else api.SLA2_F32,
                        flags=api.SLA2_FLAG_SAVE_FOR_BACKWARD)
    ws = api.alloc_workspace(p)
    api.sla2_forward(p, q, kk, v, rw, alpha, torch.empty_like(q), workspace=ws)
    got = []
    for _ in range(2):
        got.append([torch.full_like(q, float("nan")) for _ in range(3)] + [torch.full_like(alpha, float("nan"))])
        api.sla2_backward(p, q, kk, v, alpha, dout, *got[-1], ws)
    for a, b in zip(*got):
        assert torch.equal(a, b) and not torch.isnan(a).any()
