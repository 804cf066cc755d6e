"""GPU parity of the bf16 tree attention over every count of 32-key stages that its two key
groups and its ring of slots can meet in one split (256 KV heads: the plan takes one split)."""
import numpy as np
import pytest
import torch

import oracle
from tests import _util as U
from workloads import BF16, bf16_bits_to_f32, f32_to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [2, 31, 32, 33, 64, 65, 97, 129, 161, 224, 225, 257, 289, 352])
def test_one_split_of_every_stage_count(rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_00487_amd as taps
    H, N, hd, pr = 256, 2, 128, 32
    ctx = rows - N
    print(f"[attn-stages] rows={rows}", flush=True)
    rng = np.random.default_rng(rows)
    Q, K, V = (f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))
               for s in ((1, N, H, hd), (rows, H, hd), (rows, H, hd)))
    par, n = np.array([[-1, 0]], dtype=np.int32), np.array([N], dtype=np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    c = np.array([ctx], dtype=np.int32)
    att = taps.TreeAttention(1, N, H, H, hd, ctx, dtype=BF16)
    att.ws.fill_(0xFF)
    O = att(U.to_dev(Q, True), U.to_dev(K, True), U.to_dev(V, True),
            torch.zeros(1, dtype=torch.int64).cuda(), dev(c), dev(par), dev(n))
    got = U.gpu_o_as_f64(O)
    ref = oracle.tree_attention(*(bf16_bits_to_f32(a).astype(np.float64) for a in (Q, K, V)),
                                np.zeros(1, dtype=np.int64), c, list(par), [N], hd ** -0.5)
    assert not np.isnan(got).any()
    # bf16 probabilities (2^-9 each, renormalised) and a bf16 result, |O| <= max |V|
    assert np.abs(got - ref).max() <= 3 * 2.0 ** -9 * np.abs(bf16_bits_to_f32(V)).max()
    # the same rows in shuffled pages give the same bits
    pages = -(-rows // pr)
    table = rng.permutation(pages).astype(np.int32)
    Kp, Vp = (np.zeros((pages, pr, H, hd), dtype=a.dtype) for a in (K, V))
    for r in range(rows):
        Kp[table[r // pr], r % pr], Vp[table[r // pr], r % pr] = K[r], V[r]
    pat = taps.PagedTreeAttention(1, N, H, H, ctx, pr)
    pat.ws.fill_(0xFF)
    Op = pat(U.to_dev(Q, True), U.to_dev(Kp, True), U.to_dev(Vp, True), dev(table[None]), dev(c),
             dev(par), dev(n))
    assert torch.equal(O.view(torch.int16), Op.view(torch.int16))
