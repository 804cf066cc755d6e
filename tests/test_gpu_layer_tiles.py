"""GPU parity of the verification layer where its projections run in tiles of 256 and 128 rows
with the epilogue in the GEMM: ragged last tiles, a hidden size that is no multiple of 128, a
split of the grid into both tile heights, nodes past n_nodes, and the paged stores."""
import numpy as np
import pytest
import torch

from tests.test_gpu_layer import _run, taps  # noqa: F401
from workloads import kv_offsets

pytestmark = pytest.mark.gpu


def _fused(taps, B, N, H, Hq, Hkv, max_ctx):
    """Both projections fused: the scratch holds only the rotations besides Q, O and the
    attention's."""
    lib = taps.load()
    al = lambda x: (x + 255) & ~255
    rest = 2 * al(B * N * Hq * 256) + al(
        lib.tree_verify_attn_workspace_bytes(B, N, Hq, Hkv, 128, max_ctx, 0))
    return lib.verify_layer_workspace_bytes(B, N, Hq, Hkv, 128, H, max_ctx) - rest == al(B * N * 512)


@pytest.mark.parametrize("B,N,H,Hq,Hkv,both", [
    (5, 420, 832, 8, 4, True),       # 256-row tiles, the last of 52 rows; 64 columns left over
    (3, 300, 192, 16, 8, False),     # 128-row tiles, the last of 4 rows
    (5, 420, 192, 20, 5, False),     # 256 tiles of 256 rows, the others of 128
])
def test_layer_tiles(taps, B, N, H, Hq, Hkv, both):  # noqa: F811
    rng = np.random.default_rng(N + H)
    ctx = [int(rng.integers(0, 40)) for _ in range(B)]
    n = [N, N - 1, 1, 0, N][:B]
    assert _fused(taps, B, N, H, Hq, Hkv, max(ctx)) or not both
    _run(taps, rng, B, N, H, Hq, Hkv, ctx, n,
         sample_nodes=lambda b: sorted({0, n[b] // 2, max(0, n[b] - 1)} & set(range(n[b]))))


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
