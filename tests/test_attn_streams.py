"""One fp32 TreeAttention object on several streams at once: its calls share no scratch."""
import pytest
import torch

import paper_2606_00487_amd as taps
from paper_2606_00487_amd import BF16, FP32

SHAPE = (1, 32, 8, 2, 128, 2048)   # long enough to be split


def _inputs(seed, device, dtype=torch.float32):
    g = torch.Generator().manual_seed(seed)
    _, N, Hq, Hkv, hd, ctx = SHAPE
    r = lambda *s: torch.randn(*s, generator=g).to(dtype).to(device)
    parent = torch.tensor([[-1] + [(i - 1) // 2 for i in range(1, N)]], dtype=torch.int32)
    return (r(1, N, Hq, hd), r(ctx + N, Hkv, hd), r(ctx + N, Hkv, hd),
            torch.zeros(1, dtype=torch.int64, device=device),
            torch.tensor([ctx], dtype=torch.int32, device=device), parent.to(device),
            torch.tensor([N], dtype=torch.int32, device=device))


@pytest.mark.parametrize("dtype", [FP32, BF16])
def test_scratch_by_stream(monkeypatch, dtype):
    """Which scratch a call hands to the library, with the streams and the call played (host
    only): the object's own on the stream it was made on, another one on any other."""
    at = {"stream": 11}
    calls = []

    class Lib:
        @staticmethod
        def tree_verify_attn(*a):
            calls.append(a[-3:])
            return 0

    monkeypatch.setattr(taps, "_stream", lambda: at["stream"])
    monkeypatch.setattr(taps, "_need", lambda *a: None)
    monkeypatch.setattr(taps._lib, "check", lambda *a: None)
    att = taps.TreeAttention(*SHAPE, dtype=dtype, device="cpu")
    assert att.ws_bytes > 0
    att.lib, att._home = Lib, 11
    x = _inputs(0, "cpu", torch.float32 if dtype == FP32 else torch.bfloat16)
    for at["stream"] in (11, 12, 11):
        att(*x)
    assert [c[2] for c in calls] == [11, 12, 11] and {c[1] for c in calls} == {att.ws_bytes}
    assert calls[0][0] == calls[2][0] == att.ws.data_ptr()
    assert (calls[1][0] != att.ws.data_ptr()) == (dtype == FP32)


@pytest.mark.gpu
def test_fp32_attention_on_three_streams():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    att = taps.TreeAttention(*SHAPE, dtype=FP32)
    xs = [_inputs(s, "cuda") for s in range(3)]
    want = [att(*x) for x in xs]
    torch.cuda.synchronize()
    streams = [torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [[torch.zeros_like(want[0]) for _ in range(8)] for _ in xs]
    torch.cuda.synchronize()
    for rep in range(8):
        for s, x, o in zip(streams, xs, outs):
            with torch.cuda.stream(s):
                att(*x, out=o[rep])
    torch.cuda.synchronize()
    for w, o in zip(want, outs):
        for rep in range(8):
            assert torch.equal(o[rep], w), rep
