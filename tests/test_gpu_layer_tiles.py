"""GPU parity of the verification layer over the kernels that its projections' plans choose
from: tiles of 256 and 128 rows with the epilogue in the GEMM (ragged last tiles, a hidden size
that is no multiple of 128, a split of the grid into both tile heights, nodes past n_nodes, the
paged stores), the same tiles with K splits, and 64-row workgroups of every width with the
rotary pass of one and of four heads per wave.  Every case asserts the plan it is there for."""
import numpy as np
import pytest
import torch

from tests._util import layer_plans
from tests.test_gpu_layer import _run, taps  # noqa: F401
from tests.test_gpu_paged import _run_layer_paged
from workloads import kv_offsets

pytestmark = pytest.mark.gpu


def _plans(B, N, H, Hq, Hkv):
    """(K splits, output columns and rows per workgroup) of the Q/K/V and output projections."""
    return tuple((p.splits, p.cols, p.rows) for p in layer_plans(B, N, H, Hq, Hkv))


TILES = (1, 128, 256)   # 256- and 128-row tiles, the epilogue in the GEMM


@pytest.mark.parametrize("B,N,H,Hq,Hkv,oproj", [
    (5, 420, 832, 8, 4, TILES),          # 256-row tiles, the last of 52 rows; 64 columns left over
    (3, 300, 192, 16, 8, (4, 64, 64)),   # 128-row tiles, the last of 4 rows
    (5, 420, 192, 20, 5, (2, 64, 64)),   # 256 tiles of 256 rows, the others of 128
])
def test_layer_tiles(taps, B, N, H, Hq, Hkv, oproj):  # noqa: F811
    rng = np.random.default_rng(N + H)
    ctx = [int(rng.integers(0, 40)) for _ in range(B)]
    n = [N, N - 1, 1, 0, N][:B]
    assert _plans(B, N, H, Hq, Hkv) == (TILES, oproj)
    _run(taps, rng, B, N, H, Hq, Hkv, ctx, n,
         sample_nodes=lambda b: sorted({0, n[b] // 2, max(0, n[b] - 1)} & set(range(n[b]))))


# the plans that write fp32 partials, Q/K/V projection first; heads: of the rotary pass per wave
# (four from 8192 (node, head) pairs on, the last group of 10 heads partly filled)
SPLIT = [
    (4, 99, 1216, 16, 4, (1, 96, 64), (4, 128, 256), 4),    # tiles, output projection
    (4, 99, 2560, 12, 4, (4, 128, 256), (1, 128, 64), 1),   # tiles, Q/K/V projection
    (13, 64, 2560, 6, 2, (4, 128, 256), TILES, 4),
    (13, 64, 192, 6, 2, (1, 128, 64), (4, 64, 64), 4),      # 128 columns and 64 rows
    (2, 40, 1216, 12, 4, (4, 128, 64), (4, 64, 64), 1),
    (2, 40, 640, 40, 8, (1, 64, 64), (16, 128, 64), 1),
]


def _split_case(B, N, H, Hq, Hkv, qkv, oproj, heads):
    assert _plans(B, N, H, Hq, Hkv) == (qkv, oproj)
    assert (4 if B * N * (Hq + 2 * Hkv) > 8192 else 1) == heads
    rng = np.random.default_rng(B + H)
    ctx = [int(rng.integers(0, 70)) for _ in range(B)]
    n = [[N, N - 3, 1, 0, N // 2][b % 5] for b in range(B)]
    pick = lambda b: sorted({0, n[b] // 3, max(0, n[b] - 1)} & set(range(n[b])))
    return rng, ctx, n, pick


@pytest.mark.parametrize("case", SPLIT, ids=lambda c: "x".join(map(str, c[:5])))
def test_layer_plans(taps, case):  # noqa: F811
    rng, ctx, n, pick = _split_case(*case)
    _run(taps, rng, *case[:5], ctx, n, sample_nodes=pick)


@pytest.mark.parametrize("case", SPLIT[:4], ids=lambda c: "x".join(map(str, c[:5])))
def test_layer_plans_paged(taps, case):  # noqa: F811
    rng, ctx, n, pick = _split_case(*case)
    _run_layer_paged(taps, rng, *case[:5], ctx, n, 32, sample_nodes=pick)


def test_layer_tiles_paged(taps):  # noqa: F811
    B, N, H, Hq, Hkv, pr = 3, 300, 192, 16, 8, 32
    rng = np.random.default_rng(8)
    g = torch.Generator(device="cuda").manual_seed(8)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.bfloat16)
    ctx, n = np.array([33, 0, 64], np.int32), np.array([N, N - 7, 5], np.int32)
    tree = taps.TreeBuffers.empty(B, 1, 1, N)
    par = np.stack([np.r_[-1, [rng.integers(max(0, i - 9), i) for i in range(1, N)]]
                    for _ in range(B)]).astype(np.int32)
    dep = np.zeros_like(par)
    for i in range(1, N):
        dep[:, i] = dep[np.arange(B), par[:, i]] + 1
    tree.parent.copy_(torch.from_numpy(par))
    tree.depth.copy_(torch.from_numpy(dep))
    tree.n_nodes.copy_(torch.from_numpy(n))
    w = taps.LayerWeights(r(Hq * 128, H) / 14, r(Hkv * 128, H) / 14, r(Hkv * 128, H) / 14,
                          r(H, Hq * 128) / 45, r(128), r(128))
    X = r(B, N, H)
    off = kv_offsets(ctx, N)
    rows = int(off[-1] + ctx[-1] + N)
    K, V = r(rows, Hkv, 128), r(rows, Hkv, 128)
    need = [-(-int(c + N) // pr) for c in ctx]
    ids = rng.permutation(sum(need))
    table = np.zeros((B, max(need)), np.int32)
    Kp, Vp = (torch.zeros(sum(need), pr, Hkv, 128, dtype=torch.bfloat16, device="cuda")
              for _ in range(2))
    at = [(int(ids[sum(need[:b]) + j // pr]), j % pr) for b in range(B) for j in range(int(ctx[b]) + N)]
    for b in range(B):
        table[b, :need[b]] = ids[sum(need[:b]):sum(need[:b + 1])]
    pg, sl = (torch.tensor(x, device="cuda") for x in zip(*at))
    Kp[pg, sl], Vp[pg, sl] = K, V
    dev = lambda a: torch.from_numpy(a).cuda()
    Y = taps.VerifyLayer(B, N, Hq, Hkv, 128, H, int(ctx.max()))(X, w, K, V, dev(off), dev(ctx), tree)
    Yp = taps.PagedVerifyLayer(B, N, Hq, Hkv, 128, H, int(ctx.max()), pr)(X, w, Kp, Vp, dev(table),
                                                                          dev(ctx), tree)
    assert torch.equal(Kp[pg, sl], K) and torch.equal(Vp[pg, sl], V)
    for b in range(B):
        assert torch.equal(Y[b, :n[b]], Yp[b, :n[b]])
