"""The ragged work list's choice of a split length: batches of 2 to 70 requests (one wave holds
64) with lengths close together, far apart and empty, over each branch of the choice and both
sides of its limits, both head sizes, against the oracle.  bf16 outputs of bf16 probabilities:
the suite's bound of 2e-2 on values of a few units."""
import numpy as np
import pytest
import torch

import oracle
from tests import _util as U
from workloads import BF16, bf16_bits_to_f32, f32_to_bf16_bits, kv_offsets

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def taps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_00487_amd as taps
    taps.load()
    return taps


def _branch(R, max_ctx, N, Hq, Hkv, hd):
    """The branch of the choice for requests of R keys: little work, every request cut for
    max_ctx without a list ("plain"); the list with the host's length ("host"), for more requests
    than a wave has lanes ("many") or with the cheapest of 64 lengths ("search")."""
    steps = len(R) * Hkv * -(-N * (Hq // Hkv) // 128) * (max_ctx + N) // 64
    if steps < (4096 if hd == 128 else 3072):
        return "plain"
    if 4 * max(R) * len(R) <= 5 * sum(R):
        return "host"
    return "many" if len(R) > 64 else "search"


SQ70 = [(37 * i * i) % 900 for i in range(70)]
SQ64 = [(97 * i * i) % 3000 for i in range(64)]


@pytest.mark.parametrize("hd,ctx,N,Hq,Hkv,branch", [
    (hd, *c, "plain") for hd in (64, 128) for c in [
        ([3000, 5], 9, 4, 2), ([500, 510, 505], 40, 8, 2), ([0, 0], 1, 2, 1),
        ([700, 1400, 2100, 64, 0], 33, 8, 2), (SQ70, 5, 4, 1)]] + [
    (128, [6000, 40, 2500, 0], 64, 32, 8, "search"), (128, SQ64, 5, 4, 2, "search"),
    (128, SQ70, 5, 8, 8, "many"),
    (128, [4100, 2432], 64, 64, 16, "search"),   # just past the 5/4 of the mean
    (128, [4100, 2434], 64, 64, 16, "host"),     # just within it
    (128, [4032, 100], 64, 64, 16, "search"),    # 4096 steps of 64 keys
    (128, [4031, 100], 64, 64, 16, "plain"),     # one key fewer
    (64, [6200, 40, 2500, 0], 64, 32, 8, "search"), (64, SQ70, 5, 8, 8, "many"),
    (64, SQ64, 5, 8, 4, "search"), (64, [2100, 2000, 2050, 1800, 1700, 2010], 128, 32, 8, "host"),
    (64, [3008, 100], 64, 64, 16, "search"),     # 3072 steps of 64 keys
    (64, [3007, 100], 64, 64, 16, "plain"),      # one key fewer
])
def test_ragged_pick(taps, hd, ctx, N, Hq, Hkv, branch):
    rng = np.random.default_rng(len(ctx) + hd)
    B, ctx = len(ctx), np.array(ctx, dtype=np.int32)
    print(f"[ragged-pick] hd={hd} B={B} N={N} ctx={ctx.tolist()}", flush=True)
    off = kv_offsets(ctx, N)
    rows = int(off[-1] + ctx[-1] + N)
    Q, K, V = (f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))
               for s in ((B, N, Hq, hd), (rows, Hkv, hd), (rows, Hkv, hd)))
    parents = [np.array([-1] + [int(rng.integers(max(0, i - 3), i)) for i in range(1, N)],
                        dtype=np.int32) for _ in range(B)]
    n = [N if b % 3 else max(1, N - 2) for b in range(B)]
    R = [int(c) + k for c, k in zip(ctx, n)]
    assert _branch(R, int(max(ctx.max(), 1)), N, Hq, Hkv, hd) == branch
    att = taps.TreeAttention(B, N, Hq, Hkv, hd, int(max(ctx.max(), 1)), dtype=BF16)
    att.ws.fill_(0xFF)            # NaN bits in every unwritten partial slot
    O = att(U.to_dev(Q, True), U.to_dev(K, True), U.to_dev(V, True), torch.from_numpy(off).cuda(),
            torch.from_numpy(ctx).cuda(), torch.from_numpy(np.stack(parents)).cuda(),
            torch.tensor(n, dtype=torch.int32).cuda())
    torch.cuda.synchronize()
    f64 = lambda x: bf16_bits_to_f32(x).astype(np.float64)
    ref = oracle.tree_attention(f64(Q), f64(K), f64(V), off, ctx, parents, n, hd ** -0.5)
    got = U.gpu_o_as_f64(O)
    for b in range(B):
        U.attention_error(got[b, :n[b]], ref[b, :n[b]], BF16, f"pick hd={hd} b={b} ctx={ctx[b]}")
