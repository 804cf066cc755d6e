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


def _branch(R, N, Hq, Hkv):
    """The branch of the kernel's choice for requests of R keys: the host's length ("host"),
    128-key splits that all fit the 256 CUs ("short"), more requests than a wave has lanes
    ("many"), or the cheapest of 64 lengths ("search")."""
    units = Hkv * -(-N * (Hq // Hkv) // 128)
    if 4 * max(R) * len(R) <= 5 * sum(R):
        return "host"
    if len(R) > 64:
        return "many"
    return "short" if sum(-(-r // 128) for r in R) * units <= 256 else "search"


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("ctx,N,Hq,Hkv,branch", [
    ([3000, 5], 9, 4, 2, "short"), ([500, 510, 505], 40, 8, 2, "host"), ([0, 0], 1, 2, 1, "host"),
    ([700, 1400, 2100, 64, 0], 33, 8, 2, "short"),
    ([(37 * i * i) % 900 for i in range(70)], 5, 4, 1, "many"),
    ([6000, 40, 2500, 0], 64, 16, 4, "search"),
    ([(97 * i * i) % 3000 for i in range(64)], 5, 4, 1, "search"),
    ([7100, 900], 32, 8, 4, "short"),      # 64 splits of 4 units: just the chip
    ([7169, 900], 32, 8, 4, "search"),     # one split more
    ([2000, 1170], 16, 8, 8, "short"),     # just past the 5/4 of the mean
    ([2000, 1200], 16, 8, 8, "host")])     # just within it
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
    assert _branch([int(c) + k for c, k in zip(ctx, n)], N, Hq, Hkv) == branch
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
