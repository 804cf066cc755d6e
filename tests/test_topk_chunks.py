"""The vocabulary scan's chunk length on each side of its rule, read off the scratch that a call
asks for (host only): 8192 where more than 384 workgroups of 16384 would scan, but not for bf16
rows whose full-vocabulary sums are taken chunk by chunk as well."""
import ctypes

import pytest

from paper_2606_00487_amd import _lib
from paper_2606_00487_amd import BF16, FP32, LEARNED, LOGITS, MARGINAL, SIBLING


def _chunks(batch, block, vocab, K, dtype, scorer):
    buf = ctypes.create_string_buffer(256)     # stands for the scorer's arrays, never read
    at = ctypes.addressof(buf)
    mlp = _lib.ScorerMLP(at, at, at, at, 0.0, at, 16, 32)
    p = _lib.SelectParams(batch, block, vocab, K, 64, dtype, LOGITS, 1.0, 0.125, 0.0, 1.0, scorer,
                          ctypes.pointer(mlp))
    lib = _lib.load()
    assert lib.taps_select_validate(ctypes.byref(p)) == _lib.TAPS_OK
    per = 8 * K + {SIBLING: 0, MARGINAL: 32, LEARNED: 64}[scorer]
    return lib.taps_select_workspace_bytes(ctypes.byref(p)) // (batch * block * per)


@pytest.mark.parametrize("K", [4, 8, 16])
@pytest.mark.parametrize("batch,block,vocab,dtype,scorer,length", [
    (8, 16, 262144, BF16, SIBLING, 8192),
    (8, 16, 262144, BF16, MARGINAL, 16384),
    (8, 16, 262144, BF16, LEARNED, 16384),
    (8, 16, 262144, FP32, MARGINAL, 8192),
    (8, 16, 262143, BF16, MARGINAL, 8192),     # rows of the general path
    (4, 8, 196608, BF16, SIBLING, 16384),      # 384 workgroups
    (4, 8, 196616, BF16, SIBLING, 8192),       # more
    (4, 8, 196608, FP32, MARGINAL, 16384),
    (4, 8, 196609, FP32, MARGINAL, 8192),
    (16, 32, 300000, BF16, SIBLING, 16384),    # 8192 would leave more than 16384 lists
])
def test_chunk_length(batch, block, vocab, dtype, scorer, length, K):
    assert _chunks(batch, block, vocab, K, dtype, scorer) == -(-vocab // length)
