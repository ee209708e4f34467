"""The states of the key blocks that sla2_forward leaves in the workspace (bf16 tensors): K^phi as fragments, z_j, lnZ and the
totals, against fp64 on the stored K and V - in every split of the kernel over threads (d, quantisation, states of long lists)
and at the edges of its tiles."""
import numpy as np
import pytest

from paper_2602_12675_amd import workloads as W
from helpers import run_forward

pytestmark = pytest.mark.gpu


def states(inp, b, h):
    """fp64: K^phi [N, d], lnZ [N] of one head."""
    x = inp.values("k", b, h)
    x = x - x.mean(0)
    m = x.max(1, keepdims=True)
    e = np.exp(x - m)
    s = e.sum(1, keepdims=True)
    return e / s, (m + np.log(s))[:, 0]


def fragments(phi, T_n, d):
    """K^phi of whole blocks as sla2.h lays the fragments out: [T_n, d/32, 4, 64, 8]."""
    pad = np.zeros((T_n * 64, d))
    pad[:len(phi)] = phi
    mt, ks, l, i = np.meshgrid(range(d // 32), range(4), range(64), range(8), indexing="ij")
    tok, ch = 16 * ks + 8 * (i // 4) + 4 * (l // 32) + i % 4, 32 * mt + l % 32
    return pad.reshape(T_n, 64, d)[:, tok, ch]


# the block counts leave runs of one, several and unequal numbers of blocks to a workgroup
@pytest.mark.parametrize("N", [1, 63, 64, 65, 1000])
@pytest.mark.parametrize("quant", ["none", "fp8", "int8", "fp8v"])
@pytest.mark.parametrize("d", [64, 128])
def test_states_of_key_blocks(d, quant, N):
    check(W.TINY.replace(name="kv-state", dtype="bf16", quant=quant, per_head_freq=True, grid=(1, 1, N), d=d, block_q=64, H=3, B=2,
                         topk_frac=0.2))


def test_runs_of_several_blocks():
    """More blocks than workgroups: 40 heads of 17 blocks, the last of one token."""
    check(W.TINY.replace(name="kv-runs", dtype="bf16", quant="fp8", grid=(1, 1, 1025), d=128, block_q=128, H=40, topk_frac=0.1), heads=[0, 39])


@pytest.mark.parametrize("quant", ["none", "fp8v"])
def test_states_of_long_lists(quant):
    """H_i formed ahead (T_n = 128, k = 77; the last block of one token): no K^phi is kept, z_j, lnZ and the totals are."""
    check(W.TINY.replace(name="kv-long", dtype="bf16", quant=quant, grid=(1, 1, 8129), d=128, block_q=128, H=24, topk_frac=0.6),
          heads=[0, 23], phi=False)


def check(w, heads=None, phi=True):
    import torch
    from paper_2602_12675_amd import api
    inp = W.generate(w)
    r = run_forward(api, torch, inp)
    L = api.sla2_workspace_layout(r["p"])
    BH, T_n, d = w.B * w.H, w.T_n, w.d
    view = lambda off, dt, shape: api.workspace_view(r["ws"], off, dt, shape).float().cpu().numpy().astype(np.float64)
    assert (L.z_blocks > L.k_phi) == phi
    z = view(L.z_blocks, torch.float32, (BH, T_n, d))
    lnz = view(L.k_stats, torch.float32, (BH, w.N))
    h_total, z_total = view(L.h_total, torch.float32, (BH, d, d)), view(L.z_total, torch.float32, (BH, d))
    frag = view(L.k_phi, torch.bfloat16, (BH, T_n, d // 32, 4, 64, 8)) if phi else None
    for bh in range(BH) if heads is None else heads:
        p, ln = states(inp, bh // w.H, bh % w.H)
        V = inp.values("v", bh // w.H, bh % w.H)
        # fp32 exponentials of arguments below 2^4 (the tensors hold |x| < 8), whose rounding is 2^-20 at the worst on lnZ and
        # 2^-20 of an entry on K^phi; sums of 64 positive entries keep the relative error
        np.testing.assert_allclose(lnz[bh], ln, rtol=0, atol=2.0 ** -19)
        zj = np.add.reduceat(p, np.arange(0, w.N, 64), axis=0)
        np.testing.assert_allclose(z[bh], zj, rtol=2.0 ** -18, atol=0)
        np.testing.assert_allclose(z_total[bh], p.sum(0), rtol=2.0 ** -17, atol=0)
        # bf16 keeps 8 bits: half a unit in the last place is 2^-8 of an entry at most (and 2^-18 from before)
        if phi:
            np.testing.assert_allclose(frag[bh], fragments(p, T_n, d), rtol=2.0 ** -8 * 1.01, atol=0)
        # every product is off by 2^-8 of itself at most, the sums by 2^-18 of the sum of magnitudes
        assert np.all(np.abs(h_total[bh] - p.T @ V) <= 2.0 ** -8 * 1.02 * (p.T @ np.abs(V)) + 1e-30)
