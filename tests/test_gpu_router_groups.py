"""The router at the edges of its groups of 16 key blocks and its rounds of 256, and its selection with equal scores."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _route(q, k, rw, d, frac):
    import torch
    from paper_2602_12675_amd import api
    B, H, N, _ = q.shape
    p = api.make_params(B, H, N, d, 64, 64, frac, dtype=api.SLA2_BF16)
    kk = api.sla2_num_selected(p)
    t_m = -(-N // 64)
    idx = torch.full((B, H, t_m, kk), -1, dtype=torch.int32, device="cuda")
    api.sla2_router(p, q, k, rw, idx, api.alloc_workspace(p))
    torch.cuda.synchronize()
    return idx.cpu().numpy(), kk


def _expected(q, k, rw, d, kk):
    import torch
    B, H, N, _ = q.shape
    pad = -N % 64
    cnt = torch.full((-(-N // 64), 1), 64.0, dtype=torch.float64)
    cnt[-1] = 64.0 - pad
    pool = lambda x: torch.nn.functional.pad(x.double().cpu(), (0, 0, 0, pad)).reshape(B, H, -1, 64, d).sum(3) / cnt
    w = rw.double().cpu()
    s = (pool(q) @ (w[0] @ w[1].T)) @ pool(k).transpose(-1, -2)
    order = torch.sort(s, dim=-1, descending=True, stable=True).indices[..., :kk]     # equal scores: the lower index first
    return np.sort(order.numpy(), axis=-1)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("t_n", [1, 15, 16, 17, 255, 257, 529])
def test_router_group_edges(t_n, d):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(t_n)
    q, k = (torch.randn((1, 2, 64 * t_n - (t_n % 3), d), generator=gen, device="cuda").bfloat16() for _ in range(2))
    rw = torch.randn((2, d, d), generator=gen, device="cuda")
    frac = 1.0 if t_n == 1 else 0.2
    idx, kk = _route(q, k, rw, d, frac)
    assert np.array_equal(idx, _expected(q, k, rw, d, kk))


@pytest.mark.parametrize("copies", [2, 3, 40])
def test_router_equal_scores_at_the_edge(copies):
    """Every key block occurs `copies` times: whole groups of equal scores straddle the k-th place."""
    import torch
    t_n, d = 120, 64
    gen = torch.Generator(device="cuda").manual_seed(copies)
    q = torch.randn((1, 2, 64 * t_n, d), generator=gen, device="cuda").bfloat16()
    # small integers: block sums and products are exact, so that equal blocks have equal scores in every summation order
    k = torch.randint(-2, 3, (1, 2, t_n // copies, 64, d), generator=gen, device="cuda").repeat(1, 1, copies, 1, 1)
    k = k.reshape(1, 2, 64 * t_n, d).bfloat16()
    rw = torch.eye(d, device="cuda").repeat(2, 1, 1)
    idx, kk = _route(q.round(), k, rw, d, 0.1)
    assert np.array_equal(idx, _expected(q.round(), k, rw, d, kk))


@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_router_takes_the_part_of_the_workspace_that_it_uses(dtype):
    """Up to the pooled keys in `partial`; what the forward pass puts behind them (fp32: the states of all key blocks) is not asked for."""
    import torch
    from paper_2602_12675_amd import api
    B, H, N, d = 1, 3, 2048, 128
    gen = torch.Generator(device="cuda").manual_seed(4)
    q, k = (torch.randn((B, H, N, d), generator=gen, device="cuda").to(getattr(torch, dtype)) for _ in range(2))
    rw = torch.randn((2, d, d), generator=gen, device="cuda")
    p = api.make_params(B, H, N, d, 128, 64, 0.25, dtype=api.SLA2_F32 if dtype == "float32" else api.SLA2_BF16)
    whole = api.alloc_workspace(p)
    need = api.sla2_workspace_layout(p).partial + B * H * (N // 64) * d * 8
    idx, mask = [], []
    for ws in (whole, whole[:need].clone()):
        idx.append(torch.full((B, H, N // 128, 8), -1, dtype=torch.int32, device="cuda"))
        mask.append(torch.zeros((B, H, N // 128, N // 64), device="cuda"))
        api.sla2_router(p, q, k, rw, idx[-1], ws)
        api.sla2_router_soft(p, q, k, rw, 0.1, mask[-1], ws)
    assert torch.equal(idx[0], idx[1]) and torch.equal(mask[0], mask[1]) and int(idx[0].min()) >= 0
    short = whole[:need - 1]
    assert api.sla2_router(p, q, k, rw, idx[0], short, check=False) == api.SLA2_EWORKSPACE
    assert api.sla2_router_soft(p, q, k, rw, 0.1, mask[0], short, check=False) == api.SLA2_EWORKSPACE
