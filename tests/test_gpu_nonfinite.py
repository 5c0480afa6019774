"""NaN and infinity stay where they belong: a query row that holds one, a padded query or a key
that a row does not see must not change any other row. Each launch variant of the attention kernels
is run twice on the same inputs, once with the values in question finite, and the rows that may not
change are compared bit by bit (a row's arithmetic is its own: nothing of it depends on its
neighbours' values)."""
import numpy as np
import pytest
import torch

from gpu_util import dev, i32, randn
from paper_2411_01783_amd import binding as B

pytestmark = pytest.mark.gpu

# name: sizes of the ranks' queries and KV, heads, KV heads, head_dim, dtype. What they are for:
#   uncut / cut   a workgroup per unit; equal shares with a merge
#   split         more keys than the plan's table holds, few rows: KV axis over the grid
#   whole         256 row blocks in one call
#   walk          shards behind their arrival flags
#   acc           merged into a running result
#   packed        several sequences in one call
CASES = {
    "uncut": ([57, 40], [300, 211], 16, 1, 128, "bf16"),
    "cut": ([57, 340], [700, 511], 16, 2, 128, "bf16"),
    "split": ([40], [31000], 16, 1, 128, "bf16"),
    "whole": ([1040], [420], 64, 1, 128, "bf16"),
    "walk": ([1024, 1030], [500, 333], 64, 1, 128, "bf16"),
    "acc": ([1024], [500], 64, 1, 128, "bf16"),
    "packed": ([400], [400], 8, 1, 128, "bf16"),
    "cut64": ([57, 340], [700, 511], 16, 2, 64, "bf16"),
    "uncut64": ([57, 40], [300, 211], 16, 4, 64, "bf16"),
    "whole64": ([1040], [420], 64, 1, 64, "bf16"),
    "fp32": ([57, 40], [300, 211], 8, 2, 64, "fp32"),
    "fp32_128": ([57, 40], [300, 211], 8, 2, 128, "fp32"),
}


class Case:
    def __init__(self, name):
        self.name = name
        self.n_q, self.n_kv, nh, nkv, d, dtype = CASES[name]
        rng = np.random.default_rng(len(name) * 7 + d)
        t, total = sum(self.n_q), sum(self.n_kv)
        self.q = randn(5001, (t, nh, d), dtype)[0]
        self.k = randn(5002, (total, nkv, d), dtype)[0]
        self.v = randn(5003, (total, nkv, d), dtype)[0]
        if name == "packed":   # two sequences, the second from token 150 on
            self.cu = i32([0, 150, t])
            self.kv_pos = np.concatenate([np.arange(150), np.arange(total - 150)])
            self.q_pos = self.kv_pos.copy()
        else:
            # rows of a wavefront have near positions, so that some blocks are hidden from all of
            # its rows and visible to others of the workgroup
            self.kv_pos = np.arange(total)
            self.q_pos = np.sort(rng.integers(0, total, size=t))
        self.pad = [3, t // 2, t - 2]                  # padded queries
        self.q_pos[self.pad] = B.CP_POS_PAD_Q

    def run(self, out_dtype=torch.float32):
        """(O, LSE) of all tokens, with the inputs as they are now."""
        q, k, v = dev(self.q), dev(self.k), dev(self.v)
        qp, kp = i32(self.q_pos), i32(self.kv_pos)
        if self.name == "packed":
            o, l = B.cp_attn_partial(q, k, v, qp, kp, self.cu, self.cu, out_dtype=out_dtype)
        elif self.name == "acc":
            half = self.n_kv[0] // 2
            acc_o = torch.empty(q.shape, dtype=torch.float32, device="cuda")
            acc_l = torch.empty(q.shape[:2], dtype=torch.float32, device="cuda")
            o = torch.empty(q.shape, dtype=out_dtype, device="cuda")
            B.cp_attn_partial(q, k[:half].contiguous(), v[:half].contiguous(), qp, kp[:half],
                              out=acc_o, lse=acc_l)
            B.cp_attn_partial_accumulate(q, k[half:].contiguous(), v[half:].contiguous(), qp,
                                         kp[half:].clone(), acc_o, acc_l, final_out=o)
            l = acc_l
        elif len(self.n_q) == 1:
            o, l = B.cp_attn_partial(q, k, v, qp, kp, out_dtype=out_dtype)
        else:
            n = len(self.n_q)
            qs, ks = np.cumsum(self.n_q)[:-1], np.cumsum(self.n_kv)[:-1]
            cut = lambda x, at: [y.contiguous() for y in torch.tensor_split(x, at.tolist())]
            kw = {}
            if self.name == "walk":
                kw = dict(fused_merge=2, arrived=[torch.ones(n, dtype=torch.int32, device="cuda")
                                                  for _ in range(n)], spin_limit=1000)
            ring = B.Ring(cut(q, qs), cut(k, ks), cut(v, ks), cut(qp, qs), cut(kp, ks),
                          out_dtype=out_dtype, **kw)
            o, l = (torch.cat(x) for x in B.cp_ring_passkv(ring))
        torch.cuda.synchronize()
        return o.clone(), l.clone()


def same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("name", list(CASES))
def test_a_bad_query_row_stays_alone(name, value):
    c = Case(name)
    o, l = c.run()
    t, nh, d = c.q.shape
    c.q = c.q.clone()
    for tok in c.pad:                       # nothing is asked of a padded query's contents
        c.q[tok] = value
    bad = [(t // 3, 0), (t - 5, nh - 1)]
    for tok, h in bad:
        c.q[tok, h, d // 2] = value
    o2, l2 = c.run()
    keep = torch.ones((t, nh), dtype=torch.bool, device="cuda")
    for tok, h in bad:
        keep[tok, h] = False
    assert torch.isfinite(o[keep]).all()
    assert same(o2[keep], o[keep]) and same(l2[keep], l[keep])
    for tok in c.pad:
        assert (o2[tok] == 0).all() and torch.isneginf(l2[tok]).all()


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("name", list(CASES))
def test_a_hidden_bad_key_changes_nothing(name, value):
    c = Case(name)
    total = len(c.kv_pos)
    hidden = [5, 40, total // 2 + 3, total - 1]     # padded slots: no row sees them
    c.kv_pos = c.kv_pos.copy()
    c.kv_pos[hidden] = B.CP_POS_PAD_KV
    late = total - total // 4                       # a key that the later rows see
    o, l = c.run()
    c.k = c.k.clone()
    c.k[hidden] = value
    o2, l2 = c.run()
    assert torch.isfinite(o).all()
    assert same(o2, o) and same(l2, l)
    c.k[late] = value
    o2, l2 = c.run()
    blind = torch.as_tensor(c.q_pos < c.kv_pos[late]).to("cuda")
    if name == "packed":
        blind |= torch.arange(len(c.q_pos), device="cuda") < 150
    assert blind.any() and not blind.all()
    assert same(o2[blind], o[blind]) and same(l2[blind], l[blind])


# A V that a row does not see: the row is computed again, on the vector pipe and with fp32
# probabilities, so it agrees to the rounding of the path's own probabilities: none in fp32 and at
# head_dim 64 (fp32 sums of at most 2048 terms: 2^-24 sqrt(2048) of values of unit size), bf16 at
# head_dim 128. The walk behind flags asks for finite V (it has no second look).
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("name", [n for n in CASES if n != "walk"])
def test_a_hidden_bad_value_changes_nothing(name, value):
    c = Case(name)
    total = len(c.kv_pos)
    atol = 2e-2 if c.q.shape[2] == 128 and c.q.dtype == torch.bfloat16 else 1e-5
    hidden = [5, 40, total // 2 + 3, total - 1]     # padded slots: no row sees them
    c.kv_pos = c.kv_pos.copy()
    c.kv_pos[hidden] = B.CP_POS_PAD_KV
    late = total - total // 4                       # a key that the later rows see
    o, l = c.run()
    c.v = c.v.clone()
    c.v[hidden] = value
    o2, l2 = c.run()
    assert same(l2, l) and float((o2 - o).abs().max()) <= atol
    c.v[late, 0, 1] = value
    o2, l2 = c.run()
    blind = torch.as_tensor(c.q_pos < c.kv_pos[late]).to("cuda")
    if name == "packed":
        blind |= torch.arange(len(c.q_pos), device="cuda") < 150
    assert same(l2, l) and float((o2[blind] - o[blind]).abs().max()) <= atol
    assert not torch.isfinite(o2[~blind]).all()     # (the rows that see it have it)
    o3, _ = c.run(torch.bfloat16)
    assert float((o3[blind].float() - o[blind]).abs().max()) <= 2e-2
