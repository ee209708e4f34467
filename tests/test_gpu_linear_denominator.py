"""The denominator of the linear branch, Q^phi Z_i, is formed from the un-rounded fp32 Q^phi.

The input makes a rounding of Q^phi to bf16 visible: keys of two kinds, K^phi all on channel 0 with V = v_e and all on
channel 1 with V = 0, and query rows (0, x, -32, -32, ..).  With n_0, n_1 keys of the two kinds outside the selected
blocks, O_l = v_e n_0 / (n_0 + n_1 exp(x)): the numerator holds products of powers of two with v_e, exact in bf16, and
the denominator alone depends on exp(x).  The x are bf16 values whose exponential lies a quarter of a bf16 step or more
below its bf16 neighbour, so that a rounded exp(x) enlarges every denominator: by 7.6e-4 of itself or more, 1.2e-3 in
the mean.
"""
import numpy as np
import pytest

import sla2_oracle as O
from paper_2602_12675_amd import workloads as W

pytestmark = pytest.mark.gpu

SEL, BLOCKS = 1, 5                       # one selected block, four left to the linear branch: 64 + 192 keys


def _query_values():
    bits = np.arange(0x3000, 0x3F31, dtype=np.uint32).astype(np.uint16) | np.uint16(0x8000)
    x = W.bf16_bits_to_f32(bits).astype(np.float64)             # bf16 values in (-0.69, 0)
    w = np.exp(x)
    up = W.bf16_bits_to_f32(W.f32_to_bf16_bits(w.astype(np.float32))).astype(np.float64) - w
    return x[(up >= 2.0 ** -10) & (x > -0.68) & (x < -0.01)]    # a step is 2^-8 in [0.5, 1)


@pytest.mark.parametrize("frac", [0.2, 0.0], ids=["one-selected", "none-selected"])
@pytest.mark.parametrize("quant", ["none", "fp8", "int8", "fp8v"])
@pytest.mark.parametrize("d,bq", [(128, 128), (128, 64), (64, 128), (64, 64)])
def test_denominator_takes_unrounded_weights(d, bq, quant, frac):
    import torch
    from paper_2602_12675_amd import api
    N, kv = 64 * BLOCKS, 64
    if frac == 0.0:
        N = 64 * 4                                              # (256 keys outside the selection either way)
    xs = _query_values()
    assert xs.size >= 150
    rng = np.random.default_rng(d + bq)
    q = np.full((N, d), -32.0)
    q[:, 0] = 0.0
    q[:, 1] = xs[np.arange(N) % xs.size]
    first = np.arange(N) % 4 == 0                               # a quarter of the keys of every block
    k = np.zeros((N, d))
    k[np.arange(N), np.where(first, 0, 1)] = 32.0
    vals = W.bf16_bits_to_f32(W.f32_to_bf16_bits(rng.uniform(0.5, 2.0, size=d).astype(np.float32))).astype(np.float64)
    v = np.where(first[:, None], vals[None], 0.0)
    bits = [W.f32_to_bf16_bits(a.astype(np.float32))[None, None] for a in (q, k, v)]
    rw = rng.normal(size=(2, d, d)).astype(np.float32) / np.float32(np.sqrt(d))
    p = api.make_params(1, 1, N, d, bq, kv, frac, dtype=api.SLA2_BF16, quant_mode=api.QUANT_MODES[quant],
                        flags=api.SLA2_FLAG_NO_SMOOTH_K)
    assert api.sla2_num_selected(p) == (SEL if frac else 0)
    tq, tk, tv = (api.to_device(b, api.SLA2_BF16) for b in bits)
    out = torch.full_like(tq, float("nan"))
    api.sla2_forward(p, tq, tk, tv, torch.from_numpy(rw).cuda(), torch.zeros(1, device="cuda"), out, workspace=api.alloc_workspace(p))
    got = out.float().cpu().numpy()[0, 0].astype(np.float64)
    ref = vals[None] * 64.0 / (64.0 + 192.0 * np.exp(q[:, 1:2]))
    o = O.forward_head(q, k, v, rw[0].astype(np.float64), rw[1].astype(np.float64), 0.0, frac, bq, kv, smooth=False)
    np.testing.assert_allclose(o["O"], ref, rtol=1e-9)          # the closed form is what the oracle computes
    rel = got / ref - 1.0
    assert np.abs(rel).max() <= 1.01 * 2.0 ** -8                # one rounding to bf16; 1 % for a tie that fp32 decides
    # Its mean: a rounding of up to 2^-8 per output, 150 x 64 distinct quotients or more, so a standard deviation of
    # 2^-8 / sqrt(3 x 9600) = 2.3e-5 at most; six of them less what 128 fp32 sums can add (8e-6).
    assert abs(rel.mean()) <= 1.2e-4, rel.mean()
