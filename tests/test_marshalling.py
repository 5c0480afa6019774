"""The native marshalling of the binding (csrc/py_calls.cpp): what it returns and refuses, and that
other threads run while the library is called. No GPU needed."""
import ctypes
import threading

import pytest
import torch

from paper_2411_01783_amd import binding as B


def host_call(**kw):
    """cp_attn_partial without queries: checked, and returned before anything is launched."""
    a = dict(q=torch.zeros((0, 4, 128), dtype=torch.bfloat16),
             k=torch.zeros((3, 2, 128), dtype=torch.bfloat16),
             v=torch.zeros((3, 2, 128), dtype=torch.bfloat16),
             q_pos=torch.zeros(0, dtype=torch.int32), kv_pos=torch.zeros(3, dtype=torch.int32),
             workspace=torch.zeros(1 << 16, dtype=torch.uint8), stream=0)
    a.update(kw)
    return B.cp_attn_partial(**a)


def test_marshalling_returns_the_results_it_was_given():
    out = torch.zeros((0, 4, 128))
    lse = torch.zeros((0, 4))
    o, l = host_call(out=out, lse=lse)
    assert o is out and l is lse
    o, l = host_call(out_dtype=torch.float32)
    assert o.shape == (0, 4, 128) and o.dtype == torch.float32 and l.shape == (0, 4)


@pytest.mark.parametrize("kw,error", [
    (dict(q=torch.zeros((0, 4, 128), dtype=torch.float16)), TypeError),
    (dict(q=torch.zeros((0, 128), dtype=torch.bfloat16)), ValueError),
    (dict(v=torch.zeros((3, 128, 2), dtype=torch.bfloat16).transpose(1, 2)), AssertionError),
    (dict(k=torch.zeros((3, 3, 128), dtype=torch.bfloat16)), B.CpError),      # 4 heads on 3
    (dict(q=torch.zeros((0, 4, 96), dtype=torch.bfloat16)), B.CpError),
    (dict(cu_seqlens_q=torch.zeros(2, dtype=torch.int32)), B.CpError),        # one of the two
])
def test_marshalling_refuses(kw, error):
    with pytest.raises(error):
        host_call(**kw)


def test_marshalling_lets_other_threads_run():
    # one of the library's functions replaced by one that sleeps without the interpreter's lock
    native, lib = B._calls(), B.load()
    real = [ctypes.cast(getattr(lib, x), ctypes.c_void_p).value for x in
            ("cp_workspace_bytes", "cp_attn_partial", "cp_attn_decode", "cp_attn_decode_static",
             "cp_attn_merge", "cp_kv_append", "cp_ring_passkv", "cp_ring_passq",
             "cp_ring_passq_decode")]
    sleep = ctypes.cast(ctypes.CDLL(None).usleep, ctypes.c_void_p).value
    steps, stop = [0], threading.Event()

    def count():
        while not stop.wait(0.001):
            steps[0] += 1
    other = threading.Thread(target=count)
    try:
        native.connect(*(real[:6] + [sleep] + real[7:]))
        other.start()
        before = steps[0]
        assert native.ring(0, 300000, 0) == 0
        during = steps[0] - before
    finally:
        stop.set()
        other.join()
        native.connect(*real)
    assert during > 10      # of about 300; none or one if the lock is kept
