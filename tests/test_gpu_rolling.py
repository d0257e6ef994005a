"""GPU parity of the matrix-core kernel's rolling loop at the edges of its 32-key subtiles,
64-key tiles and two-tile steps, and on scores that move its exponent reference; of its
key-split form (small grids) and plain form (many heads), and of the two-branch launch of a
differential layer.

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


KEY_COUNTS = (1, 2, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 161, 191, 192, 193,
              224, 225, 256, 257, 320, 321, 385)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows", [40, 130])
def test_key_counts(D, rows):
    """Every remainder class of the key count: within a subtile, a tile, a two-tile step (one
    kv head: more than one key tile runs the key-split form)."""
    for n in KEY_COUNTS:
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


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows", [40, 130])  # two-wave and four-wave workgroups
@pytest.mark.parametrize("window,sinks", [(0, 0), (70, 5)])
def test_key_counts_many_heads(D, rows, window, sinks):
    """The plain form: more 64-row tiles than a round of key-split workgroups; three heads are
    compared."""
    H = 700
    for n in KEY_COUNTS[::3] if window else KEY_COUNTS:
        q, k, v = wl.make_shape_inputs(1, H, H, rows, n, D, seed=n)
        what = f"{H} heads keys {n} rows {rows} D{D} W{window}"
        announce(what)
        scale = 1.0 / math.sqrt(D)
        o = ef.attention_fwd(q.cuda(), k.cuda(), v.cuda(), scale=scale, causal=True,
                             window=window, sinks=sinks)
        torch.cuda.synchronize()
        for h in (0, 311, H - 1):
            one = slice(h, h + 1)
            ref = oracle.attention_ref(f64(q[:, one]), f64(k[:, one]), f64(v[:, one]), scale, True,
                                       window=window, sinks=sinks)
            err = np.abs(o[:, one].cpu().double().numpy() - ref)
            assert err.max() <= 1e-2, f"{what} head {h}: max {err.max():.3e}"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows", [24, 130])
def test_diff_pair_key_counts(D, rows):
    """Both branches in one launch (one partition). y = A1 - lambda A2 is normalised to unit
    RMS, so the bound of the branches' outputs, 2^-9 max|v| (1 + |lambda|), is divided by the
    row's RMS of y and scaled by (1 - lambda_init) |gamma|."""
    for n in KEY_COUNTS[2::4]:
        q1, q2, k1, k2, v, lam, gamma = wl.make_diff_inputs(1, 2, 1, rows, n, D, seed=n)
        what = f"diff keys {n} rows {rows} D{D}"
        announce(what)
        dev = [t.cuda() for t in (q1, q2, k1, k2, v)]
        vecs = [t.cuda() for t in lam + (gamma,)]
        o = ef.diff_attention(*dev, *vecs, wl.DIFF_LAMBDA_INIT, wl.DIFF_EPS, causal=False,
                              partition_size=64 * (n // 64 + 1))
        torch.cuda.synchronize()
        scale = 1.0 / math.sqrt(D)
        a1 = oracle.attention_ref(f64(q1), f64(k1), f64(v), scale, False)
        a2 = oracle.attention_ref(f64(q2), f64(k2), f64(v), scale, False)
        l64 = [t.double().numpy() for t in lam]
        mix = np.exp(l64[0] @ l64[1]) - np.exp(l64[2] @ l64[3]) + wl.DIFF_LAMBDA_INIT
        y = a1 - mix * a2
        rms = np.sqrt((y * y).mean(-1, keepdims=True) + wl.DIFF_EPS)
        g = gamma.double().numpy()
        ref = (1.0 - wl.DIFF_LAMBDA_INIT) * g * y / rms
        # Each branch is off by at most 2^-9 sum_j p_j |v_j| / l <= 2^-9 max|v|; the row's RMS
        # moves by no more than the same amount.
        dy = 2.0 ** -9 * float(v.float().abs().max()) * (1.0 + abs(mix))
        bound = (1.0 - wl.DIFF_LAMBDA_INIT) * np.abs(g) * (dy / rms) * (1.0 + np.abs(y) / rms)
        err = np.abs(o.cpu().double().numpy() - ref)
        assert (err <= bound + 1e-6).all(), f"{what}: {(err / (bound + 1e-6)).max():.3f} of bound"


@pytest.mark.parametrize("D", [64, 128])
def test_keys_at_the_end_of_the_largest_head(D):
    """Tiles whose byte offset inside the head is just below 2^32 (the largest head the ABI
    accepts): a window at its end against the same keys in a small tensor."""
    n, tail, rows, window = (2**31 - 1) // D, 400, 130, 200
    q, k, v = wl.make_shape_inputs(1, 1, 1, rows, tail, D, seed=5)
    announce(f"last {tail} of {n} keys D{D}")
    qd = q.cuda()
    big = []
    for t in (k, v):
        b = torch.zeros(1, 1, n, D, dtype=torch.bfloat16, device="cuda")
        b[:, :, n - tail:] = t.cuda()
        big.append(b)
    for sinks in (0, 3):
        o = ef.attention_fwd(qd, *big, causal=True, window=window, sinks=sinks)
        ks, vs = ([torch.cat([b[:, :, :sinks].cpu(), t], 2) for b, t in zip(big, (k, v))]
                  if sinks else (k, v))
        # The sink keys in front of the tail: rows see them whatever the window.
        ref = oracle.attention_ref(f64(q), f64(ks), f64(vs), 1.0 / math.sqrt(D), True,
                                   window=window, sinks=sinks)
        torch.cuda.synchronize()
        err = np.abs(o.cpu().double().numpy() - ref)
        assert err.max() <= 1e-2, f"sinks {sinks}: max {err.max():.3e}"


@pytest.mark.parametrize("B,Hkv,Sq,Skv", [(1, 8, 200, 200), (2, 8, 140, 500), (3, 8, 130, 131),
                                          (1, 16, 300, 1201), (8, 100, 70, 70)])
def test_longest_first_order(B, Hkv, Sq, Skv):
    """Causal launches over a multiple of eight kv heads visit their row tiles longest first
    over an XCD's heads; every row of every head is compared (the last shape: one head per
    batch row)."""
    D, G = 64, 2
    q, k, v = wl.make_shape_inputs(B, Hkv * G, Hkv, Sq, Skv, D, seed=Sq)
    announce(f"longest first {B} {Hkv} {Sq} {Skv}")
    bound = 2.0 ** -9 * float(v.float().abs().max()) + 1e-5
    scale = 1.0 / math.sqrt(D)
    o = ef.attention_fwd(q.cuda(), k.cuda(), v.cuda(), scale=scale, causal=True).cpu()
    for b in range(B):
        for h in (range(Hkv) if Hkv <= 16 else ((13 * b) % Hkv,)):
            hq = slice(G * h, G * h + G)
            ref = oracle.attention_ref(f64(q[b:b + 1, hq]), f64(k[b:b + 1, h:h + 1]),
                                       f64(v[b:b + 1, h:h + 1]), scale, True)
            err = np.abs(o[b:b + 1, hq].double().numpy() - ref)
            assert err.max() <= bound, f"batch {b} kv head {h}: max {err.max():.3e}"


def _rounded(q, k, v, scale, causal):
    """The attention of one kv head in float64, but for the rounding of each weight to bf16
    against the row's maximum over the keys of its first tile (64)."""
    s = torch.from_numpy(f64(q) @ f64(k).swapaxes(-1, -2)) * (scale / math.log(2.0))
    sq, skv = s.shape[-2:]
    if causal:
        s.masked_fill_(torch.ones(sq, skv).tril(skv - sq) == 0, -math.inf)
    w = torch.exp2(s - s[..., :64].max(-1, keepdim=True).values)
    assert float(w.max()) < 2.0 ** 8 / 16  # no 16 weights pass 2^8: the reference stays
    return ((w.float().bfloat16().double() @ v.double()) / w.sum(-1, keepdim=True)).numpy()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,rows,n", [(1, 64, 64), (3, 130, 47), (700, 64, 200), (700, 130, 97)])
def test_reference_of_the_first_tile(D, H, rows, n):
    """Weights are formed against the maximum of a row's first 64 keys, so that of a short row's
    largest weight nothing is lost in bf16. Against the same rounding in float64 what is left is
    fp32 arithmetic, and the few weights whose fp32 value (relative error below 2e-6) falls on the
    other side of a rounding boundary (share 2e-6 / 2^-9, an error of 2^-9 each, so
    sqrt(1e-3) 2^-9 = 6e-5 of the 2-norm). A reference 2^0.5 off gives 1.5e-3."""
    q, k, v = wl.make_shape_inputs(1, H, H, rows, n, D, seed=n)
    scale = 1.0 / math.sqrt(D)
    for causal in (False, True):
        if causal and rows > n:
            continue
        what = f"first tile {H} heads rows {rows} keys {n} D{D} {causal}"
        announce(what)
        o = ef.attention_fwd(q.cuda(), k.cuda(), v.cuda(), scale=scale, causal=causal)
        for h in {0, H // 2, H - 1}:
            ref = _rounded(q[:, h], k[:, h], v[:, h], scale, causal)
            err = o[:, h].cpu().double().numpy() - ref
            rel = np.linalg.norm(err) / np.linalg.norm(ref)
            assert rel <= 2e-4, f"{what} head {h}: {rel:.2e}"


def _moving(order, sign, n, rows, D, heads, seed):
    """q, k, v with scaled scores that follow `order` along the key axis, up to about 24."""
    q, k, v = wl.make_shape_inputs(1, 2 * heads, heads, rows, n, D, seed=seed)
    j = torch.arange(n, dtype=torch.float32)
    ramp = {"rising": j / n, "falling": 1.0 - j / n,
            "spikes": (j % 97 == 96).float()}[order][None, None, :, None]
    u = torch.randn(D, generator=torch.Generator().manual_seed(3))
    u = u / u.norm()
    q = (q.float() - (q.float() @ u)[..., None] * u + 6.0 * u).to(torch.bfloat16)
    k = (k.float() + sign * 4.0 * math.sqrt(D) * ramp * u).to(torch.bfloat16)
    return q, k, v


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows", [20, 70])  # two-wave and four-wave workgroups
@pytest.mark.parametrize("order", ["rising", "falling", "spikes"])
def test_reference_moves_plain(D, rows, order):
    """As test_reference_moves, through the plain form (many heads; three are compared)."""
    H, n = 700, 419
    q, k, v = _moving(order, 1.0, n, rows, D, H, 7)
    scale = 1.0 / math.sqrt(D)
    bound = 2.0 ** -9 * float(v.float().abs().max()) + 1e-5
    for causal in (False, True):
        what = f"{order} {H} heads rows {rows} D{D} {causal}"
        announce(what)
        o = ef.attention_fwd(q.cuda(), k.cuda(), v.cuda(), scale=scale, causal=causal).cpu()
        for h in (0, 311, H - 1):
            hq = slice(2 * h, 2 * h + 2)
            ref = oracle.attention_ref(f64(q[:, hq]), f64(k[:, h:h + 1]), f64(v[:, h:h + 1]),
                                       scale, causal)
            err = np.abs(o[:, hq].double().numpy() - ref)
            assert err.max() <= bound, f"{what} head {h}: max {err.max():.3e}"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows", [24, 130])
@pytest.mark.parametrize("order", ["rising", "falling", "spikes"])
@pytest.mark.parametrize("partition", [0, 384])  # with and without renewals of the reference
def test_reference_moves_diff(D, rows, order, partition):
    """Both branches in one launch over scores that move a branch's reference further than a
    renewal may take it down. Bound as in test_diff_pair_key_counts."""
    n = 379
    q1, k1, v = _moving(order, 1.0, n, rows, D, 1, 7)
    q2, k2, _ = _moving("falling" if order == "rising" else "rising", 1.0, n, rows, D, 1, 9)
    lam, gamma = wl.make_diff_inputs(1, 2, 1, 1, 1, D, seed=1)[5:]
    scale = 1.0 / math.sqrt(D)
    assert ef.ef_diff_attention_workspace_size(1, 2, 1, rows, n, D, partition) == 0  # one launch
    for causal in (False, True):
        what = f"diff {order} rows {rows} D{D} T{partition} {causal}"
        announce(what)
        o = ef.diff_attention(*(t.cuda() for t in (q1, q2, k1, k2, v) + tuple(lam) + (gamma,)),
                              wl.DIFF_LAMBDA_INIT, wl.DIFF_EPS, scale=scale, causal=causal,
                              partition_size=partition)
        a1 = oracle.attention_ref(f64(q1), f64(k1), f64(v), scale, causal)
        a2 = oracle.attention_ref(f64(q2), f64(k2), f64(v), scale, causal)
        l64 = [t.double().numpy() for t in lam]
        mix = np.exp(l64[0] @ l64[1]) - np.exp(l64[2] @ l64[3]) + wl.DIFF_LAMBDA_INIT
        y = a1 - mix * a2
        rms = np.sqrt((y * y).mean(-1, keepdims=True) + wl.DIFF_EPS)
        g = np.abs(gamma.double().numpy()) * (1.0 - wl.DIFF_LAMBDA_INIT)
        dy = 2.0 ** -9 * float(v.float().abs().max()) * (1.0 + abs(mix))
        ref = np.sign(gamma.double().numpy()) * g * y / rms
        err = np.abs(o.cpu().double().numpy() - ref)
        bound = g * (dy / rms) * (1.0 + np.abs(y) / rms) + 1e-6
        assert (err <= bound).all(), f"{what}: {(err / bound).max():.3f} of bound"


# B, Hq, Hkv, Sq, Skv, D: layers whose key axis the model would cut into 2 to 10 partitions.
ONE_LAUNCH = [(2, 8, 8, 40, 500, 64), (3, 12, 12, 69, 335, 128), (1, 12, 12, 128, 400, 64),
              (1, 32, 32, 1, 256, 128), (4, 16, 4, 381, 1375, 64)]


@pytest.mark.parametrize("shape", ONE_LAUNCH, ids=lambda s: "x".join(map(str, s)))
def test_diff_one_launch_is_as_precise_as_the_split(shape):
    """Where the library runs a differential layer in one launch, its error against float64 is
    that of the split it would run otherwise: the weights are rounded to bf16 against references
    taken at the same keys, so the two differ by fp32 rounding (below 1e-5, 1% of an error of
    1.5e-3) and in the vector producer's finer split of the keys (1 row), which costs the split
    nothing. A reference kept over all keys gives 1.01 (two partitions) to 1.23 (ten)."""
    B, Hq, Hkv, Sq, Skv, D = shape
    T = ef.ef_attention_splitkv_partition_size(*shape, 0)
    assert T < Skv and ef.ef_diff_attention_workspace_size(*shape, 0) == 0
    q1, q2, k1, k2, v, lam, gamma = wl.make_diff_inputs(*shape, seed=11)
    announce(f"diff precision {shape}")
    dev = [t.cuda() for t in (q1, q2, k1, k2, v) + tuple(lam) + (gamma,)]
    one, split = (ef.diff_attention(*dev, wl.DIFF_LAMBDA_INIT, wl.DIFF_EPS, causal=True,
                                    partition_size=p).cpu().double().numpy() for p in (0, T))
    ref = oracle.diff_attention_ref(f64(q1), f64(q2), f64(k1), f64(k2), f64(v), *map(f64, lam),
                                    f64(gamma), wl.DIFF_LAMBDA_INIT, wl.DIFF_EPS,
                                    1.0 / math.sqrt(D), True)
    e1, e2 = np.linalg.norm(one - ref), np.linalg.norm(split - ref)
    assert e1 <= 1.005 * e2, f"{shape}: {e1 / e2:.4f} of the split's error"


@pytest.mark.parametrize("D", [64, 128])
def test_diff_past_one_round(D):
    """More row tiles than CUs (272): the library splits the keys, bit for bit as the caller's
    own partition of that size does, and without a workspace runs one launch. The two ways differ
    by the rounding of each weight to bf16 in another place: bound as in
    test_diff_pair_key_counts, once for each."""
    B, H, Hkv, Sq, n = 1, 34, 34, 1024, 5184
    shape = (B, H, Hkv, Sq, n, D)
    q1, q2, k1, k2, v, lam, gamma = wl.make_diff_inputs(*shape, seed=13)
    announce(f"diff past one round {shape}")
    dev = [t.cuda() for t in (q1, q2, k1, k2, v)]
    vecs = [t.cuda() for t in tuple(lam) + (gamma,)]
    T = ef.splitkv_partition_size(*shape)
    assert T < n and ef.ef_diff_attention_workspace_size(*shape, 0) > 0
    args = (wl.DIFF_LAMBDA_INIT, wl.DIFF_EPS)
    chosen = ef.diff_attention(*dev, *vecs, *args, causal=True)
    assert torch.equal(chosen, ef.diff_attention(*dev, *vecs, *args, causal=True,
                                                 partition_size=T))
    o = torch.full_like(chosen, math.nan)
    ptrs = [t.data_ptr() for t in dev + [o] + vecs]
    assert ef.ef_diff_attention(*ptrs, *args, *shape, 1.0 / math.sqrt(D), True, 0, None, 0,
                                torch.cuda.current_stream().cuda_stream) == 0
    h = slice(33, 34)
    a1, a2 = (oracle.attention_ref(f64(q[:, h]), f64(k[:, h]), f64(v[:, h]), 1.0 / math.sqrt(D),
                                   True) for q, k in ((q1, k1), (q2, k2)))
    l64 = [t.double().numpy() for t in lam]
    mix = np.exp(l64[0] @ l64[1]) - np.exp(l64[2] @ l64[3]) + wl.DIFF_LAMBDA_INIT
    y = a1 - mix * a2
    rms = np.sqrt((y * y).mean(-1, keepdims=True) + wl.DIFF_EPS)
    g = gamma.double().numpy() * (1.0 - wl.DIFF_LAMBDA_INIT)
    dy = 2.0 ** -9 * float(v.float().abs().max()) * (1.0 + abs(mix))
    bound = np.abs(g) * (dy / rms) * (1.0 + np.abs(y) / rms) + 1e-6
    for got in (chosen, o):
        err = np.abs(got[:, h].cpu().double().numpy() - g * y / rms)
        assert (err <= bound).all(), f"{(err / bound).max():.3f} of bound"
    both = np.broadcast_to(bound.max(), chosen.shape)  # of every head: the same distributions
    assert (np.abs((chosen - o).cpu().double().numpy()) <= 2 * both).all()
