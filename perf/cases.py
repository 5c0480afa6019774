"""What a program on top of this library runs, as cases that can be timed.

Each case goes through the public binding (`paper_2411_01783_amd.binding`) the way a program that
serves one context-parallel rank, or simulates a whole ring on one GPU, calls it. Inputs are those
of the repository's workloads: q, k and v drawn from N(0, 1) in fp32 and rounded once, positions
from the load-balanced sharding, 16 query heads on 1 KV head of dimension 128 per GPU unless a
case says otherwise.

Kinds of case:
  decode       one rank answers one decode step: every query against its own sequence in the
               rank's packed KV (`cp_attn_decode`)
  decode_ring  one decode step of a whole ring, queries gathered (`cp_ring_passq_decode`)
  append       new K/V rows go into the persistent cache (`cp_kv_append`)
  merge        a rank combines the partial results of its ring steps (`cp_attn_merge`)
  passkv       a full prefill over all ranks of a ring (`cp_ring_passkv`)
  packed       the same for a batch of prompts of different lengths, fused
  passq        new tokens on top of a long cached context (`cp_ring_passq`)
  step         one ring step of a large prefill on its own (`cp_attn_partial`)
"""
import numpy as np
import torch

from paper_2411_01783_amd import binding as B
from paper_2411_01783_amd import workloads as W

# Tokens per sequence that an append case can take before its cache is full (a case is called
# some tens of thousands of times on one cache).
APPEND_ROOM = 49152
# Above this many rows an append starts from the same fill level in every call, as a program does
# that drops a turn and writes it again.
APPEND_REWRITE_ROWS = 32


def listed():
    return [
        # Chat-sized decode: four short conversations, the smallest attention call there is.
        dict(name="decode_chat", kind="decode", batch=4, len_lo=300, len_hi=1800, nh=16, nkv=1,
             unique=True, keep=True, out="bf16"),
        # A decode batch of 32 long sequences as one of 16 ranks sees it, called with the defaults
        # (no promise about sequence ids, results allocated by the call).
        dict(name="decode_rank_b32", kind="decode", batch=32, len_lo=2048, len_hi=8192, nh=16,
             nkv=1, unique=False, keep=False, out="bf16"),
        # The same batch over the whole ring of 16 ranks: 32K to 128K tokens a sequence.
        dict(name="decode_ring_b32", kind="decode_ring", n=16, batch=32, len_lo=32768,
             len_hi=131072, nh=16, nkv=1),
        # K/V of a decode step's tokens on their owner: 2 of 32 sequences get a token.
        dict(name="append_step", kind="append", batch=32, rows=2, nh=16, nkv=1, d=128,
             dtype="bf16"),
        # The merge at the end of a 128K prefill on one of 16 ranks: 16 fp32 partials.
        dict(name="merge_128k", kind="merge", tokens=8192, nh=16, d=128, parts=16, part="fp32",
             out="bf16"),
        # The small fp32 configuration: 512 tokens, two ranks, head dimension 64.
        dict(name="ring_fp32_512", kind="passkv", t=512, n=2, nh=4, nkv=1, d=64, dtype="fp32",
             fused=0),
        # An ordinary prompt on a model with head dimension 64 and grouped KV heads.
        dict(name="ring_d64_4k", kind="passkv", t=4096, n=4, nh=8, nkv=2, d=64, dtype="bf16",
             fused=0),
        # Prompts of different lengths prefilled together.
        dict(name="packed_prompts", kind="packed", batch=6, len_lo=200, len_hi=3000, n=4, nh=16,
             nkv=1, d=128),
        # The long prefill: 128K tokens over 16 ranks, a rank's ring in one launch.
        dict(name="ring_128k", kind="passkv", t=131072, n=16, nh=16, nkv=1, d=128, dtype="bf16",
             fused=2),
        # A short follow-up question on 128K cached tokens, queries gathered.
        dict(name="passq_128", kind="passq", t_new=128, p=131072, n=16, nh=16, nkv=1,
             gathered=True),
        # A longer follow-up, queries passed round the ring.
        dict(name="passq_1024", kind="passq", t_new=1024, p=131072, n=16, nh=16, nkv=1,
             gathered=False),
        # One ring step of a 1M-token prefill over 16 ranks.
        dict(name="step_1m", kind="step", s=65536, n=16, a=9, b=4, nh=16, nkv=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["decode", "decode_ring", "append", "merge", "fp32", "d64", "packed",
                       "passkv", "passq", "step"])
    nh, nkv = rng.choice([(16, 1), (16, 1), (8, 1), (8, 2), (16, 4)])
    if kind == "decode":
        lo = _log_int(rng, 48, 4096)
        return dict(kind="decode", batch=_log_int(rng, 1, 48), len_lo=lo,
                    len_hi=lo + _log_int(rng, 16, 4096), nh=nh, nkv=nkv,
                    unique=rng.random() < 0.6, keep=rng.random() < 0.5,
                    out=rng.choice(["bf16", "fp32"]))
    if kind == "decode_ring":
        n = rng.choice([2, 4, 8, 16])
        lo = _log_int(rng, 1024, 65536)
        return dict(kind="decode_ring", n=n, batch=n * rng.randint(1, 32 // n), len_lo=lo,
                    len_hi=lo + _log_int(rng, 64, 65536), nh=nh, nkv=nkv)
    if kind == "append":
        batch = rng.randint(1, 48)
        rows = rng.randint(1, batch) if rng.random() < 0.5 else _log_int(rng, 33, 8192)
        return dict(kind="append", batch=batch, rows=rows, nh=nh, nkv=1, d=128,
                    dtype=rng.choice(["bf16", "bf16", "fp32"]))
    if kind == "merge":
        return dict(kind="merge", tokens=_log_int(rng, 24, 8192), nh=nh, d=128,
                    parts=rng.choice([2, 3, 4, 6, 8, 12, 16]), part=rng.choice(["fp32", "bf16"]),
                    out=rng.choice(["bf16", "fp32"]))
    if kind == "fp32":
        nh, nkv = rng.choice([(4, 1), (4, 2), (8, 2)])
        return dict(kind="passkv", t=_log_int(rng, 150, 2500), n=rng.choice([1, 2, 3, 4]), nh=nh,
                    nkv=nkv, d=rng.choice([64, 64, 128]), dtype="fp32", fused=0)
    if kind == "d64":
        nh, nkv = rng.choice([(8, 1), (8, 2), (8, 8), (16, 2)])
        return dict(kind="passkv", t=_log_int(rng, 300, 6000), n=rng.choice([1, 2, 4, 8]), nh=nh,
                    nkv=nkv, d=64, dtype="bf16", fused=0)
    if kind == "packed":
        lo = _log_int(rng, 32, 2000)
        return dict(kind="packed", batch=rng.randint(2, 12), len_lo=lo,
                    len_hi=lo + _log_int(rng, 8, 3000), n=rng.choice([1, 2, 4]), nh=nh, nkv=nkv,
                    d=128)
    if kind == "passkv":
        t, n = _log_int(rng, 700, 100000), rng.choice([2, 4, 8, 16])
        whole = (t // n) * nh >= 1 << 16     # shards long enough for one launch per rank
        return dict(kind="passkv", t=t, n=n, nh=nh, nkv=nkv, d=128, dtype="bf16",
                    fused=rng.choice([0, 1, 2, 2]) if whole else 0)
    if kind == "passq":
        n = rng.choice([4, 8, 16])
        gathered = rng.random() < 0.5
        t = _log_int(rng, 64, 6000)
        t = max(1, t // (2 * n)) * 2 * n if gathered else t   # equal shards can be gathered
        return dict(kind="passq", t_new=t, p=_log_int(rng, 8192, 131072), n=n, nh=nh, nkv=nkv,
                    gathered=gathered)
    a, b = rng.randrange(16), rng.randrange(16)
    return dict(kind="step", s=_log_int(rng, 96, 40000), n=16, a=a, b=b, nh=nh, nkv=nkv)


# ---------------------------------------------------------------------------

def _dt(name):
    return W.torch_dtype(name)


def _i32(x):
    return torch.as_tensor(np.asarray(x, dtype=np.int32)).to("cuda")


def _take(t, pos):
    return t[torch.as_tensor(np.asarray(pos, dtype=np.int64)).to("cuda")].contiguous()


def _seed(seed, i):
    return (int(seed) * 1000 + i) % (1 << 62)


def _normal(seed, i, shape, dtype="bf16"):
    return W.normal(_seed(seed, i), shape, dtype, "cuda")


def _lengths(case):
    """The sequences' lengths belong to the case, not to the seed: one case is one amount of
    work."""
    rng = np.random.default_rng(case["len_lo"] * 131 + case["batch"])
    return rng.integers(case["len_lo"], case["len_hi"] + 1, size=case["batch"]).astype(np.int64)


def _prepare_decode(c, seed):
    lens = _lengths(c)
    total, batch = int(lens.sum()), c["batch"]
    cu = np.concatenate([[0], np.cumsum(lens)])
    st = dict(q=_normal(seed, 0, (batch, c["nh"], 128)),
              k=_normal(seed, 1, (total, c["nkv"], 128)),
              v=_normal(seed, 2, (total, c["nkv"], 128)),
              q_pos=_i32(lens - 1), kv_pos=_i32(np.concatenate([np.arange(n) for n in lens])),
              cu=_i32(cu), bid=_i32(np.random.default_rng(seed).permutation(batch)))
    st["q_pos"] = st["q_pos"][st["bid"].long()].contiguous()
    kw = dict(out_dtype=_dt(c["out"]))
    if c["unique"]:
        kw["unique_bid"] = True
    if c["keep"]:   # a serving loop's own result buffers and workspace
        shape = B.make_shape(B.CP_BF16, 128, c["nh"], c["nkv"], batch, total, batch,
                             flags=B.CP_SHAPE_UNIQUE_BID if c["unique"] else 0)
        kw["out"] = torch.empty((batch, c["nh"], 128), dtype=_dt(c["out"]), device="cuda")
        kw["lse"] = torch.empty((batch, c["nh"]), dtype=torch.float32, device="cuda")
        kw["workspace"] = torch.empty(B.cp_workspace_bytes(shape, B.CP_WS_DECODE) + 256,
                                      dtype=torch.uint8, device="cuda")
    st["kw"] = kw
    return st


def _run_decode(st):
    return B.cp_attn_decode(st["q"], st["k"], st["v"], st["q_pos"], st["kv_pos"], st["cu"],
                            st["bid"], **st["kw"])


def _prepare_decode_ring(c, seed):
    lens = _lengths(c)
    n, batch = c["n"], c["batch"]
    ks, vs, kps, cus = [], [], [], []
    for r in range(n):
        pos, cu = [], [0]
        for b, length in enumerate(lens):
            p = B.cp_shard_positions(int(length) - 1, n, r)
            if b % n == r:      # the rank that owns the sequence's new token
                p = np.concatenate([p, np.array([length - 1], dtype=np.int32)])
            pos.append(p)
            cu.append(cu[-1] + len(p))
        ks.append(_normal(seed, 10 + 2 * r, (cu[-1], c["nkv"], 128)))
        vs.append(_normal(seed, 11 + 2 * r, (cu[-1], c["nkv"], 128)))
        kps.append(_i32(np.concatenate(pos)))
        cus.append(_i32(cu))
    order = np.argsort(np.arange(batch) % n, kind="stable")
    per = batch // n
    q = _normal(seed, 0, (batch, c["nh"], 128))
    q_pos, bid = _i32(lens[order] - 1), _i32(order)
    sl = [slice(r * per, (r + 1) * per) for r in range(n)]
    ring = B.Ring([q[x] for x in sl], ks, vs, [q_pos[x] for x in sl], kps,
                  out_dtype=torch.float32, keep_partials=True, gathered_q=True, cu_seqlens_kv=cus,
                  bid=[bid[x] for x in sl], unique_bid=True)
    return dict(ring=ring)


def _prepare_append(c, seed):
    batch, rows = c["batch"], c["rows"]
    step = rows <= APPEND_REWRITE_ROWS
    counts = np.zeros(batch, dtype=np.int64)
    for i in range(rows):       # dealt round over the sequences
        counts[(i * 17 + 3) % batch] += 1
    cap = [int(n) * APPEND_ROOM if step else int(n) + 64 for n in counts]
    cache = B.KVCache(cap, c["nkv"], c["d"], dtype=_dt(c["dtype"]))
    shape = (rows, c["nkv"], c["d"])
    return dict(cache=cache, k=_normal(seed, 0, shape, c["dtype"]),
                v=_normal(seed, 1, shape, c["dtype"]), pos=_i32(np.arange(rows) + 1000),
                cu=_i32(np.concatenate([[0], np.cumsum(counts)])),
                used=None if step else cache.used.clone())


def _run_append(st):
    cache = st["cache"]
    if st["used"] is not None:
        cache.used.copy_(st["used"])
    B.cp_kv_append(cache, st["k"], st["v"], st["pos"], st["cu"])
    return cache.k, cache.v, cache.kv_pos, cache.used


def _prepare_merge(c, seed):
    tokens, nh = c["tokens"], c["nh"]
    outs, lses = [], []
    for s in range(c["parts"]):
        o = _normal(seed, 2 * s, (tokens, nh, c["d"]), c["part"])
        x = 8.0 + W.normal(_seed(seed, 2 * s + 1), (tokens, nh), "fp32", "cuda")
        if s % 2 == 1:          # load-balanced ring: the early half of the rows sees nothing of
            o[: tokens // 2] = 0        # every other shard
            x[: tokens // 2] = -float("inf")
        outs.append(o)
        lses.append(x)
    return dict(outs=outs, lses=lses, out_dtype=_dt(c["out"]))


def _run_merge(st):
    return B.cp_attn_merge(st["outs"], st["lses"], out_dtype=st["out_dtype"])


def _prepare_passkv(c, seed):
    t, n = c["t"], c["n"]
    q = _normal(seed, 0, (t, c["nh"], c["d"]), c["dtype"])
    k = _normal(seed, 1, (t, c["nkv"], c["d"]), c["dtype"])
    v = _normal(seed, 2, (t, c["nkv"], c["d"]), c["dtype"])
    pos = [B.cp_shard_positions(t, n, r) for r in range(n)]
    ps = [_i32(p) for p in pos]
    kw = {}
    if c["fused"] == 2:         # every shard behind its arrival flag; all of them are here
        kw["arrived"] = [torch.ones(n, dtype=torch.int32, device="cuda") for _ in range(n)]
    ring = B.Ring([_take(q, p) for p in pos], [_take(k, p) for p in pos],
                  [_take(v, p) for p in pos], ps, ps, out_dtype=_dt(c["dtype"]),
                  fused_merge=c["fused"], **kw)
    return dict(ring=ring)


def _prepare_packed(c, seed):
    lens, n = _lengths(c), c["n"]
    cu = np.concatenate([[0], np.cumsum(lens)])
    total = int(cu[-1])
    q = _normal(seed, 0, (total, c["nh"], c["d"]))
    k = _normal(seed, 1, (total, c["nkv"], c["d"]))
    v = _normal(seed, 2, (total, c["nkv"], c["d"]))
    qs, ks, vs, ps, cus = [], [], [], [], []
    for r in range(n):
        pos = [B.cp_shard_positions(int(x), n, r) for x in lens]
        rows = np.concatenate([p.astype(np.int64) + cu[b] for b, p in enumerate(pos)])
        qs.append(_take(q, rows))
        ks.append(_take(k, rows))
        vs.append(_take(v, rows))
        ps.append(_i32(np.concatenate(pos)))
        cus.append(_i32(np.concatenate([[0], np.cumsum([len(p) for p in pos])])))
    ring = B.Ring(qs, ks, vs, ps, ps, out_dtype=torch.bfloat16, cu_seqlens_q=cus,
                  cu_seqlens_kv=cus)
    return dict(ring=ring)


def _prepare_passq(c, seed):
    t, p, n = c["t_new"], c["p"], c["n"]
    q = _normal(seed, 0, (t, c["nh"], 128))
    k = _normal(seed, 1, (p + t, c["nkv"], 128))
    v = _normal(seed, 2, (p + t, c["nkv"], 128))
    qpos = [B.cp_shard_positions(t, n, r, offset=p) for r in range(n)]
    kvpos = [np.concatenate([B.cp_shard_positions(p, n, r), qpos[r]]) for r in range(n)]
    if c["gathered"]:
        q, qp = _take(q, np.concatenate(qpos) - p), _i32(np.concatenate(qpos))
        ends = np.cumsum([0] + [len(x) for x in qpos])
        qs = [q[ends[r]:ends[r + 1]] for r in range(n)]
        qps = [qp[ends[r]:ends[r + 1]] for r in range(n)]
    else:
        qs, qps = [_take(q, x - p) for x in qpos], [_i32(x) for x in qpos]
    ring = B.Ring(qs, [_take(k, x) for x in kvpos], [_take(v, x) for x in kvpos], qps,
                  [_i32(x) for x in kvpos], out_dtype=torch.bfloat16,
                  keep_partials=c["gathered"], gathered_q=c["gathered"])
    return dict(ring=ring)


def _prepare_step(c, seed):
    s, n = c["s"], c["n"]
    qp = B.cp_shard_positions(s * n, n, c["a"])
    kp = B.cp_shard_positions(s * n, n, c["b"])
    nq, nk = len(qp), len(kp)
    return dict(q=_normal(seed, 0, (nq, c["nh"], 128)), k=_normal(seed, 1, (nk, c["nkv"], 128)),
                v=_normal(seed, 2, (nk, c["nkv"], 128)), q_pos=_i32(qp), kv_pos=_i32(kp))


def _run_step(st):
    # a stored partial of the ring: fp32, as the merge reads it
    return B.cp_attn_partial(st["q"], st["k"], st["v"], st["q_pos"], st["kv_pos"],
                             out_dtype=torch.float32)


_PREPARE = dict(decode=_prepare_decode, decode_ring=_prepare_decode_ring, append=_prepare_append,
                merge=_prepare_merge, passkv=_prepare_passkv, packed=_prepare_packed,
                passq=_prepare_passq, step=_prepare_step)
_RUN = dict(decode=_run_decode, append=_run_append, merge=_run_merge, step=_run_step,
            decode_ring=lambda st: B.cp_ring_passq_decode(st["ring"]),
            passkv=lambda st: B.cp_ring_passkv(st["ring"]),
            packed=lambda st: B.cp_ring_passkv(st["ring"]),
            passq=lambda st: B.cp_ring_passq(st["ring"]))


def prepare(case, seed):
    return dict(_PREPARE[case["kind"]](case, seed), go=_RUN[case["kind"]])


def run(state):
    return state["go"](state)


# ---------------------------------------------------------------------------

def _visible(qp, kp):
    return int(np.searchsorted(np.sort(kp).astype(np.int64), qp.astype(np.int64),
                               side="right").sum())


def work(case):
    """Every input element read once, every output element written once; 4 d flops for every
    visible (query, key) pair and query head."""
    c, kind = case, case["kind"]
    nh, nkv, d = c["nh"], c.get("nkv", 1), c.get("d", 128)
    size = 4 if c.get("dtype") == "fp32" else 2

    def attention(n_q, n_kv, pairs, out_size):
        return {"bytes": n_q * nh * d * size + 2 * n_kv * nkv * d * size + 4 * (n_q + n_kv) +
                n_q * nh * (d * out_size + 4), "flops": 4 * d * nh * pairs}
    if kind == "decode":
        total = int(_lengths(c).sum())
        return attention(c["batch"], total, total, 4 if c["out"] == "fp32" else 2)
    if kind == "decode_ring":
        total = int(_lengths(c).sum())
        return attention(c["batch"], total, total, 4)
    if kind == "append":
        return {"bytes": c["rows"] * (4 * nkv * d * size + 8), "flops": 0}
    if kind == "merge":
        parts, rows = c["parts"], c["tokens"] * nh
        seen = rows * parts - (parts // 2) * (c["tokens"] // 2) * nh   # empty partials: LSE only
        psize, osize = (4 if c[x] == "fp32" else 2 for x in ("part", "out"))
        return {"bytes": seen * d * psize + rows * parts * 4 + rows * (d * osize + 4),
                "flops": 2 * seen * d}
    if kind == "passkv":
        return attention(c["t"], c["t"], c["t"] * (c["t"] + 1) // 2, size)
    if kind == "packed":
        lens = _lengths(c)
        return attention(int(lens.sum()), int(lens.sum()), int((lens * (lens + 1) // 2).sum()), 2)
    if kind == "passq":
        t, p = c["t_new"], c["p"]
        return attention(t, p + t, t * p + t * (t + 1) // 2, 2)
    qp = B.cp_shard_positions(c["s"] * c["n"], c["n"], c["a"])
    kp = B.cp_shard_positions(c["s"] * c["n"], c["n"], c["b"])
    return attention(len(qp), len(kp), _visible(qp, kp), 4)


def tolerance(case):
    if case["kind"] == "append":
        return "exact"              # a copy
    if case.get("dtype") == "fp32" or (case["kind"] == "merge" and case["part"] == "fp32" and
                                       case["out"] == "fp32"):
        return {"rel": 1e-5}        # fp32 sums
    return {"rel": 1e-2}            # bf16 inputs, probabilities or results
