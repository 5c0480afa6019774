"""Calls on another stream than torch's current one that allocate their scratch and results: the
memory belongs to that stream until its kernels have run, whatever the current stream allocates in
the meantime."""
import numpy as np
import pytest
import torch

from gpu_util import dev, i32, randn
from paper_2411_01783_amd import binding as B

pytestmark = pytest.mark.gpu


KEEP = []      # inputs outlive the kernels that read them


def kept(*tensors):
    KEEP.extend(tensors)
    torch.cuda.synchronize()
    return tensors


def inputs(tq, tk):
    return kept(*[dev(randn(6000 + i, (n, h, 128))[0]) for i, (n, h) in
            enumerate(((tq, 16), (tk, 1), (tk, 1)))], i32(np.full(tq, tk)), i32(np.arange(tk)))


def partial(stream):
    return B.cp_attn_partial(*inputs(64, 20000), out_dtype=torch.float32, stream=stream)


def accumulate(stream):
    q, k, v, qp, kp = inputs(2048, 300)
    o, l = kept(torch.zeros(q.shape, device="cuda"),
                torch.full(q.shape[:2], -float("inf"), device="cuda"))
    B.cp_attn_partial_accumulate(q, k, v, qp, kp, o, l, stream=stream)
    return o, l


def decode(stream, unique):
    q, k, v, _, kp = inputs(4, 9000)
    cu, qp, bid = kept(i32([0, 1000, 4000, 4100, 9000]), i32([9000] * 4), i32(np.arange(4)))
    return B.cp_attn_decode(q, k, v, qp, kp, cu, bid, out_dtype=torch.float32,
                            stream=stream, unique_bid=unique)


def merge(stream):
    parts = kept(*[randn(6100 + i, (3000, 16, 128), "fp32")[0].to("cuda") for i in range(3)])
    lses = kept(*[randn(6200 + i, (3000, 16), "fp32")[0].to("cuda") for i in range(3)])
    return B.cp_attn_merge(parts, lses, stream=stream)


CALLS = dict(partial=partial, accumulate=accumulate, decode=lambda s: decode(s, False),
             decode_unique=lambda s: decode(s, True), merge=merge)


@pytest.mark.parametrize("raw", [False, True])
@pytest.mark.parametrize("name", list(CALLS))
def test_memory_of_a_call_on_another_stream(name, raw, monkeypatch):
    want = [x.clone() for x in CALLS[name](None)]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    ours = []
    made = B._elsewhere        # the call's inputs are there: its kernels queue behind 10 ms of waiting

    def wait_there(stream, like):
        with torch.cuda.stream(side):
            torch.cuda._sleep(20_000_000)
        return made(stream, like)
    monkeypatch.setattr(B, "_elsewhere", wait_there)
    got = CALLS[name](side.cuda_stream if raw else side)
    # the current stream asks for memory of every size and fills it while the kernels wait
    for size in [1 << i for i in range(9, 27)] * 2:
        ours.append(torch.full((size,), 255, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    KEEP.clear()
    for a, b in zip(got, want):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
