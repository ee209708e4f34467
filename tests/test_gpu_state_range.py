"""States of the linear branch at the ends of what they hold: sums that cancel to a small part of their terms, sums near the largest
fp32 value, infinite entries - for long bf16 lists (H_i and dH_j as masked products of bf16 operands) and for fp32 tensors."""
import numpy as np
import pytest

import sla2_oracle as O
from helpers import rel_l2

pytestmark = pytest.mark.gpu


def call(q, k, v, frac, alpha, block_q=128, dout=None, flags=0):
    """q, k, v [1, H, N, d] on the GPU -> out, block lists (and dv for dout), the router being the identity.  H_i of bf16 tensors is a
    masked product where the lists are long and the heads many enough to fill the GPU, so some tests repeat one head."""
    import torch
    from paper_2602_12675_amd import api
    _, H, N, d = q.shape
    p = api.make_params(1, H, N, d, block_q, 64, frac, dtype=api.SLA2_BF16 if q.dtype == torch.bfloat16 else api.SLA2_F32,
                        flags=flags | (api.SLA2_FLAG_SAVE_FOR_BACKWARD if dout is not None else 0))
    rw = torch.eye(d, device="cuda").repeat(2, 1, 1)
    al = torch.full((H,), alpha, device="cuda")
    ws, out = api.alloc_workspace(p), torch.empty_like(q)
    idx = torch.empty((1, H, -(-N // block_q), api.sla2_num_selected(p)), dtype=torch.int32, device="cuda")
    api.sla2_forward(p, q, k, v, rw, al, out, block_idx=idx, workspace=ws)
    if dout is None:
        return out, idx.cpu().numpy()
    dq, dk, dv = (torch.empty_like(q) for _ in range(3))
    api.sla2_backward(p, q, k, v, al, dout, dq, dk, dv, torch.empty_like(al), ws)
    return out, idx.cpu().numpy(), dv


def test_cancelling_states():
    """H_i = (128 x 129/128 - 129 + 2^-9) h with the terms in turn: 2^-9 of h is left of 257 terms of its size.  A state held to
    2^-18 of itself would leave 128 x 2^-19 x 2^9 = 0.1 of that (its errors are the same in all terms of a sign); fp32 states
    and sums leave 2^-24 of about two terms now and then, 1e-3.  K^phi, Q^phi, H_i and the output are rounded to bf16: 2e-3 each."""
    import torch
    d, H, sel, rest = 128, 10, 90, 258
    blocks, N = sel + rest, 64 * (sel + rest)
    gen = torch.Generator().manual_seed(3)
    k0, u = torch.randn((64, d), generator=gen), torch.randint(0, 2, (64, d), generator=gen) * 2.0 - 1.0
    toward = torch.randn((d,), generator=gen)
    scale = torch.tensor([0.0] * sel + [129 / 128, -1.0] * 128 + [-1.0, 2.0 ** -9])
    k = k0 + (torch.arange(blocks) < sel)[:, None, None] * toward
    v = scale[:, None, None] * u
    q = torch.randn((N, d), generator=gen) + toward
    q, k, v = (x.reshape(1, 1, N, d).to(torch.bfloat16) for x in (q, k, v))
    out, idx = call(*(x.cuda().repeat(1, H, 1, 1) for x in (q, k, v)), sel / blocks, 0.0)
    assert (idx == np.arange(sel)).all()
    q, k, v = (x[0, 0].double().numpy() for x in (q, k, v))
    some = [0, 77, idx.shape[2] - 1]
    ref, _, _ = O.linear_branch(q, O.smooth_k(k), v, idx[0, 0], 128, 64, q_blocks=some)
    rows = np.concatenate([np.arange(128 * i, min(N, 128 * i + 128)) for i in some])
    for h in (0, H - 1):
        assert rel_l2(out[0, h].float().cpu().numpy()[rows], ref[rows]) < 1e-2


# A channel that takes nearly all of Q^phi and K^phi: H_i and dH_j are then about the number of tokens times one value.
def one_channel(N, d, gen):
    import torch
    x = 0.1 * torch.randn((N, d), generator=gen)
    x[:, 0] += 20.0
    return x


def test_large_states():
    """H_i of 1.9e38, where fp32 ends at 3.4e38."""
    import torch
    from paper_2602_12675_amd import api
    N, H, d, frac, v0 = 10240, 20, 128, 68 / 160, 3.2e34
    gen = torch.Generator().manual_seed(5)
    q, k = one_channel(N, d, gen), one_channel(N, d, gen)
    v = v0 * (1.0 + 0.1 * torch.randn((N, d), generator=gen))
    q, k, v = (x.reshape(1, 1, N, d).to(torch.bfloat16) for x in (q, k, v))
    out, idx = call(*(x.cuda().repeat(1, H, 1, 1) for x in (q, k, v)), frac, 0.25, flags=api.SLA2_FLAG_NO_SMOOTH_K)
    Q, K, V = (x[0, 0].double().numpy() for x in (q, k, v))
    some = [0, 40, 79]
    ref = O.forward_head(Q, K, V / v0, np.eye(d), np.eye(d), 0.25, frac, 128, 64, smooth=False, sel=idx[0, 0], q_blocks=some)
    rows = np.concatenate([np.arange(128 * i, 128 * i + 128) for i in some])
    for h in (0, H - 1):
        assert rel_l2(out[0, h].double().cpu().numpy()[rows] / v0, ref["O"][rows]) < 1e-2


@pytest.mark.parametrize("d,block_q,dtype", [(128, 128, "bfloat16"), (64, 64, "bfloat16"), (128, 128, "float32")])
def test_large_gradient_states(d, block_q, dtype):
    import torch
    from paper_2602_12675_amd import api
    N, frac, g0 = 2048, 0.2, 2.0e38
    gen = torch.Generator().manual_seed(6)
    q, k = one_channel(N, d, gen), one_channel(N, d, gen)
    dout = torch.zeros((N, d))
    dout[:, 5] = g0
    q, k, dout = (x.reshape(1, 1, N, d).to(getattr(torch, dtype)) for x in (q, k, dout))
    _, idx, dv = call(q.cuda(), k.cuda(), torch.zeros_like(q).cuda(), frac, 0.0, block_q, dout.cuda(), api.SLA2_FLAG_NO_SMOOTH_K)
    g = O.backward_head(q[0, 0].double().numpy(), k[0, 0].double().numpy(), np.zeros((N, d)), idx[0, 0], 0.0,
                        dout[0, 0].double().numpy() / g0, block_q, 64, smooth=False)
    assert g["dV"].max() > 0.86                        # x g0: more than half of what fp32 holds
    assert rel_l2(dv[0, 0].double().cpu().numpy() / g0, g["dV"]) < 1e-2


INFINITE = [   # H, T_n, d, block_q, type, kept fraction: both forms of the bf16 forward pass, the three of the fp32 one
    (32, 97, 128, 128, "bfloat16", 0.68), (1, 97, 128, 128, "bfloat16", 0.2), (1, 45, 128, 128, "float32", 0.2),
    (1, 97, 64, 64, "float32", 0.011), (1, 13, 64, 128, "float32", 0.3),
]


@pytest.mark.parametrize("which", ["last", "middle"])
@pytest.mark.parametrize("H,T_n,d,block_q,dtype,frac", INFINITE)
def test_infinite_value(H, T_n, d, block_q, dtype, frac, which):
    """One infinite entry of V: query blocks that did not select its key block have +inf in that channel, and what they had in
    the others; those that did have something infinite or NaN there, and what they had in the others."""
    import torch
    N, e = 64 * T_n - 7, 3
    gen = torch.Generator(device="cuda").manual_seed(8)
    q, k, v = (torch.randn((1, 1, N, d), generator=gen, device="cuda").to(getattr(torch, dtype)).repeat(1, H, 1, 1) for _ in range(3))
    plain, idx = call(q, k, v, frac, 0.5, block_q)
    j = T_n - 1 if which == "last" else idx[0, 0, 0, idx.shape[3] // 2]
    v[0, :, 64 * j, e] = float("inf")
    out, again = call(q, k, v, frac, 0.5, block_q)
    assert (idx == again).all()
    listed = np.repeat((idx[0, 0] == j).any(axis=1), block_q)[:N]
    assert not listed.all()
    others = np.arange(d) != e
    for h in (0, H - 1):
        got, want = out[0, h].double().cpu().numpy(), plain[0, h].double().cpu().numpy()
        assert np.array_equal(got[:, others], want[:, others])
        assert np.isposinf(got[~listed, e]).all() and not np.isfinite(got[listed, e]).any()


@pytest.mark.parametrize("d,block_q,dtype", [(128, 128, "bfloat16"), (64, 64, "bfloat16"), (128, 128, "float32"), (64, 64, "float32")])
@pytest.mark.parametrize("which", ["last", "middle"])
def test_infinite_gradient(d, block_q, dtype, which):
    """One infinite entry of dO in a query block: dV of the keys that it did not select is infinite in that channel alone."""
    import torch
    N, e = 2048 - 7, 3
    gen = torch.Generator(device="cuda").manual_seed(9)
    q, k, v, dout = (torch.randn((1, 1, N, d), generator=gen, device="cuda").to(getattr(torch, dtype)) for _ in range(4))
    _, idx, plain = call(q, k, v, 0.2, 0.5, block_q, dout)
    T_m = idx.shape[2]
    i = T_m - 1 if which == "last" else T_m // 2
    dout[0, 0, block_q * i, e] = float("inf")
    _, again, dv = call(q, k, v, 0.2, 0.5, block_q, dout)
    assert (idx == again).all()
    listed = np.repeat(np.isin(np.arange(-(-N // 64)), idx[0, 0, i]), 64)[:N]
    got, want = dv[0, 0].double().cpu().numpy(), plain[0, 0].double().cpu().numpy()
    others = np.arange(d) != e
    assert np.array_equal(got[~listed][:, others], want[~listed][:, others])
    assert np.isposinf(got[~listed, e]).all()


@pytest.mark.parametrize("d,block_q", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_gradients_of_the_linear_branch_for_large_queries(d, block_q):
    """Q^phi of rows up to 2^40: softmax takes differences, so all is finite and as far from fp64 as for small ones (2e-2, as the other
    gradients of bf16 tensors; d alpha sums terms of both signs).  No block selected: the scores of such rows mean nothing in fp32."""
    import torch
    from paper_2602_12675_amd import api
    N = 333
    gen = torch.Generator(device="cuda").manual_seed(9)
    q, k, v, go = (torch.randn((1, 1, N, d), generator=gen, device="cuda") for _ in range(4))
    q[:, :, 5:] *= 2.0 ** 40                         # (a few rows of ordinary size beside them)
    q, k, v, go = (x.bfloat16() for x in (q, k, v, go))
    p = api.make_params(1, 1, N, d, block_q, 64, 0.0, dtype=api.SLA2_BF16, flags=api.SLA2_FLAG_SAVE_FOR_BACKWARD)
    ws, al, da = api.alloc_workspace(p), torch.full((1,), 0.25, device="cuda"), torch.full((1,), float("nan"), device="cuda")
    dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(3))
    api.sla2_forward(p, q, k, v, torch.eye(d, device="cuda").repeat(2, 1, 1), al, torch.empty_like(q), workspace=ws)
    api.sla2_backward(p, q, k, v, al, go, dq, dk, dv, da, ws)
    Q, K, V, dO = (x[0, 0].double().cpu().numpy() for x in (q, k, v, go))
    g = O.backward_head(Q, K, V, np.zeros((-(-N // block_q), 0), dtype=np.int64), 0.25, dO, block_q, 64)
    for name, x in (("dQ", dq), ("dK", dk), ("dV", dv)):
        assert rel_l2(x[0, 0].float().cpu().numpy(), g[name]) < 2e-2, name
    assert abs(da.item() - g["dalpha"].sum()) <= 3e-2 * np.abs(g["dalpha"]).sum()


@pytest.mark.parametrize("d,block_q", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_gradients_of_the_linear_branch_near_the_largest_number(d, block_q):
    """One entry of V makes (1 - alpha) H_i dO as large as 2^127 / 3: dQ, which is a small part of it, is what a V of 2^-100 of that gives,
    times 2^100 - exact in the inputs, so a few ulp of bf16 in the result (other sums underflow there) - and finite."""
    import torch
    from paper_2602_12675_amd import api
    N = 64
    gen = torch.Generator(device="cuda").manual_seed(12)
    q, k = (torch.randn((1, 1, N, d), generator=gen, device="cuda").bfloat16() for _ in range(2))
    k[0, 0, 7, :] = 0
    k[0, 0, 7, 3] = 30.0                             # K^phi of token 7 is channel 3
    p = api.make_params(1, 1, N, d, block_q, 64, 0.0, dtype=api.SLA2_BF16, flags=api.SLA2_FLAG_SAVE_FOR_BACKWARD)
    al, rw, da = torch.zeros((1,), device="cuda"), torch.eye(d, device="cuda").repeat(2, 1, 1), torch.empty((1,), device="cuda")
    go, got = torch.ones_like(q), []
    for e in (125, 25):
        v, ws = torch.zeros_like(q), api.alloc_workspace(p)
        v[0, 0, 7, 0] = 1.25 * 2.0 ** e
        dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(3))
        api.sla2_forward(p, q, k, v, rw, al, torch.empty_like(q), workspace=ws)
        api.sla2_backward(p, q, k, v, al, go, dq, dk, dv, da, ws)
        got.append(dq[0, 0].double() * 2.0 ** -e)
    assert got[0].isfinite().all() and got[1].abs().max() > 1e-6
    assert ((got[0] - got[1]).norm() <= 2.0 ** -6 * got[1].norm()).item()
