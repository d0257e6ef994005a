"""GPU parity of the vector split producer with 3 and 4 rows per kv head, on both sides of the
workgroup count at which a partition gets one wave instead of four, and at partitions that
leave some of the four waves without a key. Tolerance: every weight is rounded to bf16
(relative 2^-9) for the value sums while the row sum adds the fp32 weights, so
|o - ref| <= 2^-9 sum_j p_j |v_j| / l <= 2^-9 max|v|, and fp32 rounding (1e-5)."""

import math

import numpy as np
import pytest
import torch

import oracle
from paper_2609_12330_amd import ef_attention as ef
from paper_2609_12330_amd import workloads as wl
from test_gpu_parity import _gpu, announce, f64  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

# B, Hq, Hkv, Sq, Skv, T, window, sinks
CASES = [
    (2, 32, 8, 1, 64 * 32, 64, 0, 0),        # 512 workgroups: four waves
    (2, 32, 8, 1, 64 * 32 + 1, 64, 0, 0),    # 528: one wave
    (2, 24, 8, 1, 64 * 31 + 17, 64, 0, 0),   # 3 rows, ragged last partition, four waves
    (2, 24, 8, 1, 64 * 33 + 17, 64, 0, 0),   # 3 rows, one wave
    (1, 4, 1, 1, 64 * 65, 64, 0, 0),         # 65 partitions: separate combine, four waves
    (1, 4, 2, 2, 700, 128, 0, 0),            # two query positions
    (2, 8, 2, 1, 3000, 256, 900, 5),         # window and sinks
] + [(1, 4, 1, 1, n, 64, 0, 0) for n in (1, 4, 5, 8, 9, 16, 17, 32, 33, 63, 64, 65)]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_decode_waves(case, D):
    B, Hq, Hkv, Sq, Skv, T, window, sinks = case
    what = f"decode waves {case} D{D}"
    announce(what)
    q, k, v = wl.make_shape_inputs(B, Hq, Hkv, Sq, Skv, D, seed=Skv)
    bound = 2.0 ** -9 * float(v.float().abs().max()) + 1e-5
    causal = Sq > 1 or window > 0
    scale = 1.0 / math.sqrt(D)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    ref = oracle.attention_ref(f64(q), f64(k), f64(v), scale, causal, window=window, sinks=sinks)
    ws = ef.make_workspace(qd, kd, T, window, sinks)
    for _ in range(2):  # the second call finds the counters the first one left
        o = ef.attention_splitkv(qd, kd, vd, scale=scale, causal=causal, partition_size=T,
                                 workspace=ws, window=window, sinks=sinks)
        torch.cuda.synchronize()
        err = np.abs(o.cpu().double().numpy() - ref)
        assert err.max() <= bound, f"{what}: max {err.max():.3e}"
    if window == 0:  # channel slices repeat the unsplit sums bit for bit
        d = ef.attention_decode_dsplit(qd, kd, vd, scale=scale, causal=causal, d_splits=2,
                                       partition_size=T)
        torch.cuda.synchronize()
        if Skv > T:
            assert torch.equal(d, o), what
