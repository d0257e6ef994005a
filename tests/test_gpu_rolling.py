"""GPU parity of the matrix-core kernel's rolling loop at the edges of its 32-key subtiles,
64-key tiles and two-tile steps, and on scores that move its exponent reference.

Tolerance: every weight is rounded to bf16 (relative 2^-9) for the value product while the
row sum adds the fp32 weights, so |o - ref| <= 2^-9 sum_j p_j |v_j| / l plus fp32 rounding,
at most 2^-9 max|v| < 1e-2 for the |v| < 5.1 drawn here.
"""

import math

import numpy as np
import pytest
import torch

import oracle
from paper_2609_12330_amd import ef_attention as ef
from paper_2609_12330_amd import workloads as wl
from test_gpu_parity import _gpu, announce, f64  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _check(q, k, v, scale, causal, what, window=0, sinks=0):
    announce(what)
    assert float(v.float().abs().max()) < 5.1
    ref = oracle.attention_ref(f64(q), f64(k), f64(v), scale, causal, window=window, sinks=sinks)
    o = ef.attention_fwd(q.cuda(), k.cuda(), v.cuda(), scale=scale, causal=causal, window=window,
                         sinks=sinks)
    torch.cuda.synchronize()
    err = np.abs(o.cpu().double().numpy() - ref)
    assert err.max() <= 1e-2, f"{what}: max {err.max():.3e}"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows", [40, 130])  # two-wave and four-wave workgroups
def test_key_counts(D, rows):
    """Every remainder class of the key count: within a subtile, a tile, a two-tile step."""
    for n in (1, 2, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 161, 191, 192, 193,
              224, 225, 256, 257, 320, 321):
        q, k, v = wl.make_shape_inputs(1, 2, 1, rows // 2, n, D, seed=n)
        for causal in (False, True):
            _check(q, k, v, 1.0 / math.sqrt(D), causal, f"keys {n} rows {rows} D{D} {causal}")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("window,sinks", [(1, 0), (33, 0), (64, 1), (65, 33), (100, 64),
                                          (160, 65)])
def test_window_edges(D, window, sinks):
    q, k, v = wl.make_shape_inputs(1, 4, 2, 150, 421, D, seed=window)
    _check(q, k, v, 1.0 / math.sqrt(D), True, f"W{window} S{sinks} D{D}", window, sinks)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("order", ["rising", "falling", "spikes"])
def test_reference_moves(D, sign, order):
    """Scores that grow along the key axis (the reference moves on many subtiles), shrink
    (never again), or jump at single keys; the weights' sums pass the move threshold."""
    n = 419
    q, k, v = wl.make_shape_inputs(1, 2, 1, 140, n, D, seed=7)
    j = torch.arange(n, dtype=torch.float32)
    ramp = {"rising": j / n, "falling": 1.0 - j / n,
            "spikes": (j % 97 == 96).float()}[order][None, None, :, None]
    u = torch.randn(D, generator=torch.Generator().manual_seed(3))
    u = u / u.norm()
    # q.u = 6 for every row, k.u rises to 4 sqrt(D): scaled scores up to about 24.
    q = (q.float() - (q.float() @ u)[..., None] * u + 6.0 * u).to(torch.bfloat16)
    k = (k.float() + sign * 4.0 * math.sqrt(D) * ramp * u).to(torch.bfloat16)
    for causal in (False, True):
        _check(q, k, v, sign / math.sqrt(D), causal, f"{order} {sign} D{D} {causal}")
