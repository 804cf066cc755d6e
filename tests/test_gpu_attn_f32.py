"""GPU parity of the fp32 tree attention (matrix-instruction kernel, split keys) against the
fp64 oracle, at the edges of its 16-row and 16-key tiles."""
import numpy as np
import pytest
import torch

import oracle
from workloads import FP32, kv_offsets

pytestmark = pytest.mark.gpu


def _case(seed, N, Hq, Hkv, hd, ctx, n):
    rng = np.random.default_rng(seed)
    B = len(ctx)
    ctx = np.array(ctx, dtype=np.int32)
    off = kv_offsets(ctx, N)
    rows = int(off[-1] + ctx[-1] + N)
    Q = rng.standard_normal((B, N, Hq, hd)).astype(np.float32)
    K = rng.standard_normal((rows, Hkv, hd)).astype(np.float32)
    V = rng.standard_normal((rows, Hkv, hd)).astype(np.float32)
    par = np.stack([np.array([-1] + [int(rng.integers(max(0, i - 9), i)) for i in range(1, N)])
                    for _ in range(B)]).astype(np.int32)
    return Q, K, V, off, ctx, par, np.array(n, dtype=np.int32)


def _run(taps, case, hd, scratch=True):
    Q, K, V, off, ctx, par, n = case
    B, N, Hq, _ = Q.shape
    att = taps.TreeAttention(B, N, Hq, K.shape[1], hd, int(ctx.max()), dtype=FP32)
    split = att.ws_bytes > 0
    if scratch:
        att.ws.fill_(0xFF)                        # NaN bits in every part not written
    else:
        att.ws, att.ws_bytes = torch.empty(16, dtype=torch.uint8, device="cuda"), 0
    O = torch.zeros(Q.shape, dtype=torch.float32, device="cuda")
    att(*(torch.from_numpy(a).cuda() for a in (Q, K, V, off, ctx, par, n)), out=O)
    torch.cuda.synchronize()
    return O.cpu().numpy().astype(np.float64), split


def _check(got, case, hd):
    Q, K, V, off, ctx, par, n = case
    ref = oracle.tree_attention(Q.astype(np.float64), K.astype(np.float64), V.astype(np.float64),
                                off, ctx, list(par), list(n), hd ** -0.5)
    # a score's sum of hd products and the exponent's three roundings, each at most 2^-24 of
    # |q| |k| / sqrt(hd), move every weight (and their sum); |O| is at most max |V|
    smax = (np.linalg.norm(Q, axis=-1).max() * np.linalg.norm(K, axis=-1).max()) * hd ** -0.5
    tol = 2 * (hd + 3) * 2.0 ** -24 * smax * np.abs(V).max()
    for b in range(len(ctx)):
        assert not np.isnan(got[b, :n[b]]).any()
        assert np.abs(got[b, :n[b]] - ref[b, :n[b]]).max(initial=0.0) <= tol
        assert not got[b, n[b]:].any()            # rows past n are not written


@pytest.fixture(scope="module")
def taps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_00487_amd as taps
    taps.load()
    return taps


@pytest.mark.parametrize("N,Hq,Hkv,hd,ctx,n", [
    (1, 1, 1, 64, [0], [1]),                      # one query, its own row alone
    (5, 3, 3, 128, [16, 11], [5, 4]),             # G = 1, a tile that ends at the tree rows
    (16, 4, 2, 64, [256, 15, 0], [16, 16, 7]),    # whole row tiles
    (17, 8, 2, 128, [2047, 33], [17, 0]),         # one row past a tile, an empty request
    (33, 40, 8, 64, [4000], [33]),                # G = 5, several splits
    (12, 4, 2, 128, [9001, 130], [12, 12]),       # many splits, more waves than tiles in one
    (130, 4, 4, 64, [700], [127]),                # masks past 64 nodes
])
def test_fp32_attention_tiles(taps, N, Hq, Hkv, hd, ctx, n):
    case = _case(N + hd, N, Hq, Hkv, hd, ctx, n)
    got, split = _run(taps, case, hd)
    print(f"[attn-f32] N={N} heads={Hq}/{Hkv} hd={hd} ctx={ctx} split={split}", flush=True)
    _check(got, case, hd)
    if split:                                     # no scratch: one split, the same result
        _check(_run(taps, case, hd, scratch=False)[0], case, hd)


def test_fp32_attention_leaves_out_hidden_rows_that_are_not_finite(taps):
    """NaN and infinities in tree rows outside a node's mask do not reach the node, and do
    reach the nodes that see them."""
    hd, ctx, N = 128, 300, 40
    case = _case(3, N, 8, 2, hd, [ctx], [N])
    Q, K, V, off, _, par, _ = case
    par[0] = np.array([-1] + [0] * (N - 1))       # a star: every node sees the root and itself
    _, split = _run(taps, case, hd)
    V[ctx + 7], V[ctx + 20, :, 3], K[ctx + 11] = np.nan, np.inf, np.nan
    for scratch in (True, False) if split else (True,):
        got = _run(taps, case, hd, scratch)[0][0]
        assert np.isnan(got[7]).all() and np.isnan(got[11]).all()
        assert np.isposinf(got[20, :, 3]).all() and np.isfinite(np.delete(got[20], 3, -1)).all()
        rest = [i for i in range(N) if i not in (7, 11, 20)]
        clean = _case(3, N, 8, 2, hd, [ctx], [N])
        clean[5][0] = par[0]
        ref = oracle.tree_attention(*(a.astype(np.float64) for a in clean[:3]), off,
                                    clean[4], list(clean[5]), [N], hd ** -0.5)[0]
        assert np.abs(got[rest] - ref[rest]).max() <= 1e-4
