"""The learned scorer's two routes, bit for bit: the rows' tables in the workspace (a row per
workgroup) and a workspace of the least size (a request per workgroup), over one row and many,
K of 1 to 16, more units than a chunk holds, rows of NaN and -inf; and the noalloc call, whose
scratch may or may not hold the tables."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def taps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_00487_amd as taps
    taps.load()
    return taps


def _weights(taps, rng, B, V, d, h):
    dev = lambda x: torch.from_numpy(np.asarray(x, dtype=np.float32)).cuda()
    F = 2 * d + 3
    return taps.ScorerWeights(
        emb=dev(rng.standard_normal((V, d)) * 0.5), W1=dev(rng.standard_normal((h, F)) * F ** -0.5),
        b1=dev(rng.standard_normal(h) * 0.1), w2=dev(rng.standard_normal(h) * h ** -0.5), b2=0.05,
        root_token=torch.from_numpy(rng.integers(0, V, B).astype(np.int32)).cuda())


FIELDS = ("parent", "token", "depth", "rank", "n_nodes", "topk_idx", "q_reach", "topk_val")


def _bits(t):
    view = {torch.float64: torch.int64, torch.float32: torch.int32}
    return {f: getattr(t, f).view(view.get(getattr(t, f).dtype, torch.int32)).clone()
            for f in FIELDS}


@pytest.mark.parametrize("B,D,V,K,N,d,h", [
    (1, 1, 40, 1, 4, 1, 1), (2, 1, 300, 16, 64, 32, 64), (3, 2, 2049, 5, 40, 7, 9),
    (1, 16, 151936, 8, 64, 16, 32), (2, 32, 5000, 8, 200, 32, 64), (2, 28, 999, 16, 300, 32, 64),
    (1300, 4, 1000, 16, 24, 8, 12)])
@pytest.mark.parametrize("special", [False, True])
def test_routes_agree(taps, B, D, V, K, N, d, h, special):
    rng = np.random.default_rng(B + V)
    x = rng.standard_normal((B, D, V)).astype(np.float32) * 3
    if special:
        x[:, D - 1] = np.nan
        x[0, 0, K // 2:] = -np.inf
    print(f"[learned-rows] B={B} D={D} V={V} K={K} d={d} h={h} special={special}", flush=True)
    m = torch.from_numpy(x).cuda().bfloat16()
    sel = taps.Selector(B, D, V, K, N, dtype=taps.BF16, scorer=taps.LEARNED,
                        mlp=_weights(taps, rng, B, V, d, h))
    assert sel.ws.numel() > sel.ws_bytes
    sel.ws.fill_(0xFF)
    full = _bits(sel(m))
    sel.ws = torch.full((sel.ws_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    least = _bits(sel(m))
    assert sel.ws_bytes <= taps._lib.SELECT_SCRATCH_BYTES
    got = taps.TreeBuffers.empty(B, D, K, N)
    sel.noalloc(m, got)
    noalloc = _bits(got)
    for f in FIELDS:
        assert torch.equal(full[f], least[f]), f
        assert torch.equal(full[f], noalloc[f]), f
