"""fp32 top-K lists against a stable sort: rows off the 16-byte alignment, chunks that the
row's end cuts, rows of one element per lane and fewer, ties past the compaction limit, both
zeros, infinities and NaN (below -inf), chunk lengths of every size."""
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


def _reference(x, K):
    key = np.where(np.isnan(x), -np.inf, x).astype(np.float64) + 0.0
    nan = np.isnan(x)
    return np.stack([np.lexsort((np.arange(x.shape[1]), -key[r], nan[r]))[:K]
                     for r in range(x.shape[0])])


@pytest.mark.parametrize("B,D,V,K", [(1, 1, 16, 16), (1, 2, 63, 8), (2, 3, 255, 4),
                                     (1, 2, 2047, 8), (1, 2, 2050, 16), (3, 5, 4097, 7),
                                     (1, 16, 151936, 8), (2, 16, 100001, 16), (16, 32, 9001, 8)])
@pytest.mark.parametrize("mode", ["normal", "ties", "special"])
def test_topk_f32(taps, B, D, V, K, mode):
    rng = np.random.default_rng(V + K)
    x = rng.standard_normal((B * D, V)).astype(np.float32)
    if mode == "ties":
        x = np.round(x).astype(np.float32) * np.where(rng.random(x.shape) < 0.5, 1, -1).astype(np.float32)
    if mode == "special":
        u = rng.random(x.shape)
        x[u < 0.3] = np.nan
        x[(u > 0.3) & (u < 0.9)] = -np.inf
        x[(u > 0.9) & (u < 0.9005)] = np.inf
        x[0] = np.nan
        x[-1, : V // 2] = -0.0
        x[-1, V // 2:] = 0.0
    print(f"[topk-f32] B={B} D={D} V={V} K={K} {mode}", flush=True)
    sel = taps.Selector(B, D, V, K, 8, dtype=taps.FP32)
    tree = sel(torch.from_numpy(x.reshape(B, D, V)).cuda())
    got = tree.topk_idx.cpu().numpy().reshape(B * D, K)
    want = _reference(x, K)
    assert np.array_equal(got, want)
    val = tree.topk_val.cpu().numpy().reshape(B * D, K)
    assert np.array_equal(val, np.take_along_axis(x, want, 1), equal_nan=True)
