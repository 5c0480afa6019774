"""GPU parity at the edges of the launch rules: which kernel or work split a call gets depends on
its sizes, and these are the sizes on either side of each rule.

Against the fp64 oracle, with the tolerances of gpu_util (2e-2 max-abs on O and 1e-3 on LSE for bf16
inputs of unit scale, 1e-4 and 1e-5 for fp32): they bound the rounding of the products and of the
probabilities whatever the split, but a key left out or counted twice among a few thousand stays
below them. So the rules of the attention launches are also taken with keys of zero
(check_counts): every visible key then has the same weight, LSE is the logarithm of their number
and O the share of each class of keys, and both come out exact, so that a single key is seen."""
import numpy as np
import pytest
import torch

from gpu_util import LSE_RTOL_FP32, O_ATOL_FP32, check, dev, i32, randn, rel_l2
from paper_2411_01783_amd import binding as B

pytestmark = pytest.mark.gpu


def ring_case(seed, kv_sizes, q_sizes, nh, nkv, d, dtype="bf16"):
    """Ring whose KV shards hold the positions 0 .. in runs in random order, and whose queries stand
    at random positions (some padded), dealt out over the ranks."""
    rng = np.random.default_rng(seed)
    total, t = sum(kv_sizes), sum(q_sizes)
    k, k64 = randn(seed + 1, (total, nkv, d), dtype)
    v, v64 = randn(seed + 2, (total, nkv, d), dtype)
    q, q64 = randn(seed + 3, (t, nh, d), dtype)
    # runs of 48 positions in random order: blocks that are visible, hidden and cut by the mask
    runs = [np.arange(a, min(a + 48, total)) for a in range(0, total, 48)]
    order = np.concatenate([runs[i] for i in rng.permutation(len(runs))])
    kv_pos = np.split(order, np.cumsum(kv_sizes)[:-1])
    q_all = np.sort(rng.integers(-1, total, size=t))
    rows = np.split(rng.permutation(t), np.cumsum(q_sizes)[:-1])
    rows = [np.sort(r) for r in rows]
    args = ([dev(q[r]) for r in rows], [dev(k[p]) for p in kv_pos], [dev(v[p]) for p in kv_pos],
            [i32(q_all[r]) for r in rows], [i32(p) for p in kv_pos])
    return args, rows, kv_pos, q_all, (q64, k64, v64)


def check_ring(oracle, ring, out, lse, case, keep, atol=2e-2, rtol=1e-3):
    _, rows, kv_pos, q_all, (q64, k64, v64) = case
    ref_o, ref_l = oracle.attn(q64, k64, v64, q_all, np.arange(len(k64)))
    for a, r in enumerate(rows):
        check(out[a], lse[a], ref_o[r], ref_l[r], atol, rtol, "merged rank %d" % a)
        if not keep:
            continue
        for b, p in enumerate(kv_pos):
            if len(r) == 0:
                continue
            po, pl = ring.partial(a, b)
            if len(p) == 0:
                assert torch.isneginf(pl).all() and (po == 0).all()
                continue
            o, l = oracle.attn(q64[r], k64[p], v64[p], q_all[r], p)
            check(po, pl, o, l, atol, rtol, "partial %d, %d" % (a, b))


def counts_case(kv_sizes, q_sizes, nh, nkv, d, q_pos, cu=None):
    """Zero keys; the value of key j is 1 in channel (j // 32 + j) % d, so that O tells which
    blocks and which keys in them were counted."""
    total, t = sum(kv_sizes), sum(q_sizes)
    pos = np.arange(total)
    k = torch.zeros((total, nkv, d), dtype=torch.bfloat16, device="cuda")
    v = torch.zeros((total, nkv, d), dtype=torch.bfloat16, device="cuda")
    cls = (pos // 32 + pos) % d
    v[torch.arange(total), :, torch.as_tensor(cls)] = 1.0
    q, _ = randn(4900, (t, nh, d))
    cut = lambda x, n: [y.contiguous() for y in torch.tensor_split(x, np.cumsum(n)[:-1].tolist())]
    args = (cut(dev(q), q_sizes), cut(k, kv_sizes), cut(v, kv_sizes), cut(i32(q_pos), q_sizes),
            cut(i32(pos), kv_sizes))
    return args, cls


def check_counts(out, lse, q_pos, cls, d, lo=0, hi=None):
    """Every row saw exactly the keys lo <= j < hi with j <= its position. Sums of ones are exact in
    fp32; the division and the logarithm err by a few 2^-24 of their result, below half a key for
    the at most 2^17.3 keys here (LSE below 12: 2^17.3 * 12 * 2^-24 is 0.12)."""
    hi = len(cls) if hi is None else hi
    classes = np.zeros((hi - lo + 1, d))
    classes[1:] = np.cumsum(np.eye(d)[cls[lo:hi]], 0)
    n = np.clip(np.asarray(q_pos) + 1 - lo, 0, hi - lo)
    ref = torch.as_tensor(classes[n], device="cuda")[:, None, :]
    nt = torch.as_tensor(n, device="cuda")[:, None]
    got = out.double() * nt[..., None].double()
    assert float((got - ref).abs().max()) < 0.5
    seen = (nt > 0).expand(lse.shape)
    assert torch.equal(torch.isneginf(lse), ~seen)
    err = (torch.exp(lse.double()) - nt.double()).abs()[seen]
    assert err.numel() == 0 or float(err.max()) < 0.5


# One rank against one shard, the sizes on either side of each rule: tiles 2 and 3, 6 and 7; row
# blocks 4 per tile; 85 and 86 with 15 and 16 tiles, 127 and 128, 255 and 256 row blocks; 512 and 513
# blocks of a split KV axis, 960 and 961 of the plan; queries that all see the same keys (left whole),
# that see everything or little (cut), in order.
@pytest.mark.parametrize("tq,tk,nh,nkv,d", [
    (30, 256, 8, 2, 128), (30, 257, 8, 2, 128), (300, 768, 16, 1, 128), (300, 769, 16, 1, 128),
    (383, 768, 16, 1, 128), (385, 768, 16, 1, 128), (2032, 769, 64, 4, 64), (2050, 640, 16, 4, 64),
    (1360, 2048, 16, 1, 128), (1361, 1920, 16, 1, 128), (1361, 2017, 16, 1, 128),
    (2032, 900, 16, 1, 128), (2033, 900, 16, 1, 128), (4080, 800, 16, 1, 128),
    (4081, 800, 16, 1, 128), (1500, 2500, 8, 8, 64), (4081, 800, 16, 1, 64),
    (70, 16384, 16, 1, 128), (70, 16385, 16, 1, 64), (600, 30720, 64, 4, 128),
    (600, 30721, 64, 4, 128), (1, 5000, 3, 1, 128),
])
def test_single_call_launch_rules_count_every_key(tq, tk, nh, nkv, d):
    rng = np.random.default_rng(tq + tk)
    half = np.where(np.arange(tq) < tq // 2, 40, tk)
    for q_pos in (np.full(tq, tk // 2), half, np.sort(rng.integers(-1, tk, size=tq))):
        args, cls = counts_case([tk], [tq], nh, nkv, d, q_pos)
        o, l = B.cp_attn_partial(*(x[0] for x in args), out_dtype=torch.float32)
        torch.cuda.synchronize()
        check_counts(o, l, q_pos, cls, d)


# Rings in one launch: the sizes of test_ring_launch_rules.
@pytest.mark.parametrize("kv_sizes,q_sizes,nh,nkv,d", [
    ([768, 0], [97, 1], 16, 1, 128), ([800, 1], [97, 2], 16, 1, 128), ([769, 31], [40, 57], 16, 1, 64),
    ([15360, 15360], [33, 16], 4, 1, 128), ([15361, 15360], [33, 16], 4, 1, 128),
    ([10239, 10273, 10209], [8, 0, 41], 8, 2, 64), ([1500, 0, 33, 1], [0, 300, 1, 17], 3, 1, 128),
    ([2000, 2100], [2000, 2080], 16, 1, 128), ([2000, 2100], [2000, 2090], 16, 1, 128),
])
def test_ring_launch_rules_count_every_key(kv_sizes, q_sizes, nh, nkv, d):
    total, t = sum(kv_sizes), sum(q_sizes)
    rng = np.random.default_rng(total + t)
    ends = np.concatenate([[0], np.cumsum(kv_sizes)])
    for q_pos in (np.full(t, total // 2), np.sort(rng.integers(-1, total, size=t))):
        args, cls = counts_case(kv_sizes, q_sizes, nh, nkv, d, q_pos)
        for keep in (False, True):
            ring = B.Ring(*args, out_dtype=torch.float32, keep_partials=keep)
            out, lse = B.cp_ring_passkv(ring)
            torch.cuda.synchronize()
            check_counts(torch.cat(out), torch.cat(lse), q_pos, cls, d)
            if not keep:
                continue
            rows = np.split(q_pos, np.cumsum(q_sizes)[:-1])
            for a, r in enumerate(rows):
                for b in range(len(kv_sizes)):
                    if len(r) > 0:
                        check_counts(*ring.partial(a, b), r, cls, d, ends[b], ends[b + 1])


# Shards kept apart, cut into parts, with few queries: parts and shards merged in one launch (up to 64
# parts in all: 14 of each of 3 shards, 16 of 4, 8 of 8, 4 and 2 of 16) and in two (13 of 5, 16 of 8);
# ranks without queries, shards that not every query sees. The result is Equation 4 over what the slots
# hold, bit by bit, whatever their type and in however many launches.
@pytest.mark.parametrize("kv_sizes,q_sizes,nh,nkv,d", [
    ([10400, 10401, 10000], [5, 0, 20], 16, 1, 128), ([8000] * 4, [9, 9, 9, 9], 16, 1, 64),
    ([4000] * 8, [8] * 8, 16, 4, 128), ([2000] * 16, [0, 8] * 8, 16, 1, 128),
    ([2000] * 16, [8] * 16, 16, 1, 64), ([6300] * 5, [3] * 5, 16, 1, 128),
    ([4000] * 8, [4] * 8, 16, 1, 128),
])
def test_kept_shards_cut_into_parts_count_every_key(kv_sizes, q_sizes, nh, nkv, d):
    total, t = sum(kv_sizes), sum(q_sizes)
    rng = np.random.default_rng(total + t)
    ends = np.concatenate([[0], np.cumsum(kv_sizes)])
    q_pos = np.sort(rng.integers(-1, total, size=t))
    args, cls = counts_case(kv_sizes, q_sizes, nh, nkv, d, q_pos)
    rows = np.split(q_pos, np.cumsum(q_sizes)[:-1])
    kept = {}
    for part in (torch.float32, torch.bfloat16):
        ring = B.Ring(*args, out_dtype=torch.float32, part_dtype=part, keep_partials=True)
        out, lse = B.cp_ring_passkv(ring)
        torch.cuda.synchronize()
        kept[part] = [[ring.partial(a, b) for b in range(len(kv_sizes))] for a in range(len(rows))]
        if part == torch.float32:
            check_counts(torch.cat(out), torch.cat(lse), q_pos, cls, d)
        messages = B.Ring(*args, out_dtype=torch.float32, part_dtype=part, keep_partials=True,
                          message_layout=True)
        out_m, lse_m = B.cp_ring_passkv(messages)
        for a, r in enumerate(rows):
            if len(r) == 0:
                continue
            for ring_, o, l in ((ring, out[a], lse[a]), (messages, out_m[a], lse_m[a])):
                slots = [ring_.partial(a, b) for b in range(len(kv_sizes))]
                want_o, want_l = B.cp_attn_merge(*zip(*slots), out_dtype=torch.float32)
                assert torch.equal(o, want_o) and torch.equal(l, want_l)
            if part == torch.float32:
                for b in range(len(kv_sizes)):
                    check_counts(*ring.partial(a, b), r, cls, d, ends[b], ends[b + 1])
    for a in range(len(rows)):
        for b in range(len(kv_sizes)):
            (o32, l32), (o16, l16) = kept[torch.float32][a][b], kept[torch.bfloat16][a][b]
            assert torch.equal(o32.to(torch.bfloat16), o16) and torch.equal(l32, l16)


# Head_dim 128 holds a probability to one bf16 term relative to the largest score of the first block of
# its piece, so results depend on where a list is cut, and that is between tiles of four blocks. Here the
# third block of every tile has keys of weight 3/2, the others of weight 1: relative to 1 both are exact
# in 8 bits, relative to 3/2 a weight of 2/3 is not (2e-3 off). The score is held in two bf16 terms, to
# 2^-17, the sums in fp32.
@pytest.mark.parametrize("kv_sizes,q_sizes,keep,packed", [
    ([15872], [20], False, 0), ([4096], [70], False, 0), ([9600], [300], False, 0),
    ([5120] * 8, [10] * 8, True, 0), ([3584] * 16, [16] * 16, True, 0), ([20480] * 3, [40, 0, 9], False, 0),
    ([1280, 1408], [400, 420], False, 3), ([2176], [900], False, 2), ([640] * 4, [200] * 4, False, 6),
])
def test_lists_are_cut_between_tiles(kv_sizes, q_sizes, keep, packed):
    batch, d, nh = max(1, packed), 128, 16
    x = np.log(1.5)
    hi = torch.tensor(x, dtype=torch.bfloat16)
    lo = torch.tensor(x - float(hi), dtype=torch.bfloat16)
    n = sum(kv_sizes)
    third = torch.arange(n, device="cuda") // 32 % 4 == 2
    k = torch.zeros((n, 1, d), dtype=torch.bfloat16, device="cuda")
    v = torch.zeros_like(k)
    k[third, :, 0], k[third, :, 1] = hi.cuda(), lo.cuda()
    v[~third, :, 0], v[third, :, 1] = 1.0, 1.0
    q = torch.zeros((sum(q_sizes), nh, d), dtype=torch.bfloat16, device="cuda")
    q[..., :2] = 1.0
    pos, q_pos = torch.arange(n, dtype=torch.int32, device="cuda"), i32(np.full(len(q), n))
    # (packed: `batch` such sequences in every shard)
    cut = lambda y, m: [torch.cat([z] * batch).contiguous()
                        for z in torch.tensor_split(y, np.cumsum(m)[:-1].tolist())]
    cu = lambda m: [i32(np.arange(batch + 1) * z) for z in m] if packed else None
    ring = B.Ring(cut(q, q_sizes), cut(k, kv_sizes), cut(v, kv_sizes), cut(q_pos, q_sizes),
                  cut(pos, kv_sizes), out_dtype=torch.float32, keep_partials=keep, softmax_scale=1.0,
                  cu_seqlens_q=cu(q_sizes), cu_seqlens_kv=cu(kv_sizes))
    out, lse = B.cp_ring_passkv(ring)
    torch.cuda.synchronize()
    ref = torch.zeros(d, device="cuda")
    ref[0], ref[1] = 2 / 3, 1 / 3
    assert float((torch.cat(out) - ref).abs().max()) < 1e-5
    assert float((torch.cat(lse) - np.log(n * 1.125)).abs().max()) < 2e-5


# A workgroup per row block over several ranks, the late chunks first: row blocks with rows of two
# chunks, of two ranks, a last one that is short; shards of one length and of others.
@pytest.mark.parametrize("kv_sizes,q_sizes,nh,nkv,d", [
    ([10400, 10401, 10000], [1501, 1500, 1499], 16, 1, 128), ([8000] * 4, [1111] * 4, 16, 1, 64),
    ([30000, 900], [700, 1401], 32, 2, 128), ([2000] * 16, [270] * 16, 16, 1, 128),
])
def test_rings_of_whole_row_blocks_count_every_key(kv_sizes, q_sizes, nh, nkv, d):
    total, t = sum(kv_sizes), sum(q_sizes)
    q_pos = np.sort(np.random.default_rng(total + t).integers(-1, total, size=t))
    args, cls = counts_case(kv_sizes, q_sizes, nh, nkv, d, q_pos)
    ring = B.Ring(*args, out_dtype=torch.float32)
    for o in ring.out:
        o.fill_(float("nan"))
    out, lse = B.cp_ring_passkv(ring)
    torch.cuda.synchronize()
    check_counts(torch.cat(out), torch.cat(lse), q_pos, cls, d)


# The last tile of a list ends after two blocks where no more than two have keys: one to five blocks,
# cut lists (parts, equal shares) that end either way, a second chunk of one and of three blocks, and a
# packed batch.
@pytest.mark.parametrize("tq,tk,nh,d", [
    (20, 32, 16, 128), (20, 64, 16, 64), (20, 65, 16, 128), (20, 96, 16, 64), (20, 129, 16, 128),
    (70, 8192 + 64, 16, 128), (70, 8192 + 65, 16, 64), (2100, 2080, 16, 128), (2100, 2112, 16, 64),
    (20, 16384 + 30, 16, 128), (20, 16384 + 96, 16, 64),
])
def test_tiles_of_two_blocks_count_every_key(tq, tk, nh, d):
    rng = np.random.default_rng(tq + tk)
    for q_pos in (np.full(tq, tk), np.sort(rng.integers(-1, tk, size=tq))):
        args, cls = counts_case([tk], [tq], nh, 1, d, q_pos)
        o, l = B.cp_attn_partial(*(x[0] for x in args), out_dtype=torch.float32)
        torch.cuda.synchronize()
        check_counts(o, l, q_pos, cls, d)
        # as two sequences of one packed batch: the same lists one after the other
        if d == 128 and tk < 4096:
            two = [torch.cat([x[0], x[0]]) for x in args]
            cu = [i32([0, n, 2 * n]) for n in (tq, tk)]
            o, l = B.cp_attn_partial(*two, out_dtype=torch.float32, cu_seqlens_q=cu[0],
                                     cu_seqlens_kv=cu[1])
            torch.cuda.synchronize()
            check_counts(o[:tq], l[:tq], q_pos, cls, d)
            check_counts(o[tq:], l[tq:], q_pos, cls, d)


# Equal shares of several units, whose rows are asked for one unit ahead: row blocks with rows of many
# ranks (some without any), the last row block short, the step from one KV head to the next, row blocks
# longer than a chunk (of 180, 181 and 255 rows).
@pytest.mark.parametrize("kv_sizes,q_sizes,nh,nkv,d", [
    ([2000, 0, 33, 1], [1, 7, 0, 300], 16, 1, 128),
    ([1500, 700], [700, 33], 12, 3, 128),
    ([40] * 31 + [900], [3, 0, 16, 1, 90, 0, 0, 5] * 4, 16, 2, 128),
    ([1500, 700], [1100, 1], 8, 4, 64),
    ([1100], [2049], 16, 4, 64),
    ([361] * 8, [361] * 8, 8, 8, 64), ([700, 0, 90, 400], [300, 0, 40, 511], 8, 8, 64),
])
def test_shares_of_units_that_hold_rows_of_many_ranks(kv_sizes, q_sizes, nh, nkv, d):
    n = max(len(kv_sizes), len(q_sizes))
    kv_sizes, q_sizes = kv_sizes + [0] * (n - len(kv_sizes)), q_sizes + [0] * (n - len(q_sizes))
    tq, tk = sum(q_sizes), sum(kv_sizes)
    rng = np.random.default_rng(tq + tk)
    for q_pos in (np.arange(tq) * tk // tq, np.sort(rng.integers(-1, tk, size=tq))):
        args, cls = counts_case(kv_sizes, q_sizes, nh, nkv, d, q_pos)
        ring = B.Ring(*args, out_dtype=torch.float32)
        out, lse = B.cp_ring_passkv(ring)
        torch.cuda.synchronize()
        check_counts(torch.cat(out), torch.cat(lse), q_pos, cls, d)


# Which workgroup runs where (xcd_slice), with every output and partial full of NaN before, so that a
# row block that nobody takes shows. Row blocks x parts of all shards. Kept apart and alike: 8 x 32 (1
# and 2 KV heads, head_dim 64), 8 x 30 of two classes, 12 x 20 of four, 12 x 18; as dispatched: a shard
# longer than the rest, 64 x 4, more than a round (84 x 4). Merged in the launch: 4 x 64, 12 x 20, 8 x 30,
# 20 x 12, and 64 x 4 as dispatched.
@pytest.mark.parametrize("kv_sizes,total_q,nh,nkv,d,keep", [
    ([8192] * 16, 128, 16, 1, 128, True), ([65536 + 33, 65536], 64, 32, 2, 64, True),
    ([43692] * 3, 126, 16, 1, 128, True), ([8213] * 4, 192, 16, 1, 128, True),
    ([5500, 5511] * 3, 192, 16, 1, 128, True), ([8192] * 15 + [16384], 128, 16, 1, 128, True),
    ([131072, 1, 0, 0], 128, 16, 4, 128, True), ([40000] * 3 + [11073], 64, 16, 1, 128, True),
    ([32768] * 4, 1024, 16, 4, 128, True), ([40000] * 4, 672, 32, 1, 128, True),
    ([10101] * 4, 68, 8, 2, 128, False), ([30000, 1, 0, 5000], 352, 8, 2, 128, False),
    ([8500] * 4, 100, 16, 4, 64, False), ([10900] * 4, 588, 8, 2, 128, False),
    ([16384] * 4, 1024, 16, 1, 128, False),
])
def test_shards_placed_on_xcds_count_every_key(kv_sizes, total_q, nh, nkv, d, keep):
    n, total = len(kv_sizes), sum(kv_sizes)
    q_sizes = [total_q // n] * n
    q_pos = np.sort(np.random.default_rng(n + total_q).integers(-1, total, size=total_q))
    args, cls = counts_case(kv_sizes, q_sizes, nh, nkv, d, q_pos)
    ring = B.Ring(*args, out_dtype=torch.float32, keep_partials=keep)
    for x in [ring.partial_out, ring.partial_lse] + ring.out + ring.lse:
        x.fill_(float("nan"))
    ring.workspace.fill_(255)
    out, lse = B.cp_ring_passkv(ring)
    torch.cuda.synchronize()
    check_counts(torch.cat(out), torch.cat(lse), q_pos, cls, d)
    ends = np.concatenate([[0], np.cumsum(kv_sizes)])
    for a, r in enumerate(np.split(q_pos, n)):
        for b in range(n if keep else 0):
            check_counts(*ring.partial(a, b), r, cls, d, ends[b], ends[b + 1])


# one shard in parts: 8 x 32 and 4 x 64 placed, 40 x 6 and three rounds (192 x 4) as dispatched
@pytest.mark.parametrize("tq,tk,nh,nkv", [
    (128, 131072, 16, 1), (64, 131072, 16, 1), (128, 131041, 16, 4), (640, 8000, 16, 1),
    (49152, 49152, 1, 1),
])
def test_parts_placed_on_xcds_count_every_key(tq, tk, nh, nkv):
    q_pos = np.sort(np.random.default_rng(tq).integers(-1, tk, size=tq))
    args, cls = counts_case([tk], [tq], nh, nkv, 128, q_pos)
    shape = B.make_shape(B.CP_BF16, 128, nh, nkv, tq, tk)
    ws = torch.full((B.cp_workspace_bytes(shape, B.CP_WS_PARTIAL) + 256,), 255, dtype=torch.uint8,
                    device="cuda")
    out = torch.full((tq, nh, 128), float("nan"), device="cuda")
    lse = torch.full((tq, nh), float("nan"), device="cuda")
    B.cp_attn_partial(*(x[0] for x in args), out=out, lse=lse, workspace=ws)
    torch.cuda.synchronize()
    check_counts(out, lse, q_pos, cls, 128)


# kv sizes, query sizes, heads, kv heads, d:
#   six tiles a unit (a workgroup per unit) and seven (equal shares, cut and merged)
#   960 blocks (bounds in LDS) and 961 (KV axis split over the grid), shards merged and kept apart
#   an empty shard, a rank without queries, a last block of one key, groups of 1, 3 and 64 heads
@pytest.mark.parametrize("kv_sizes,q_sizes,nh,nkv,d", [
    ([768], [97], 16, 1, 128),
    ([800], [97], 16, 1, 128),
    ([769, 31], [40, 57], 16, 1, 64),
    ([15360, 15360], [33, 16], 4, 1, 128),
    ([15361, 15360], [33, 16], 4, 1, 128),
    ([10239, 10273, 10209], [8, 0, 41], 8, 2, 64),
    ([1500, 0, 33, 1], [0, 300, 1, 17], 3, 1, 128),
    ([1000, 1057], [100, 31], 6, 2, 64),
    ([130, 999], [257, 3], 5, 5, 128),
    ([640, 321], [64, 5], 64, 1, 128),
])
@pytest.mark.parametrize("keep", [False, True])
def test_ring_launch_rules(oracle, kv_sizes, q_sizes, nh, nkv, d, keep):
    n = max(len(kv_sizes), len(q_sizes))
    kv_sizes = kv_sizes + [0] * (n - len(kv_sizes))
    case = ring_case(4100 + n, kv_sizes, q_sizes, nh, nkv, d)
    ring = B.Ring(*case[0], out_dtype=torch.float32, keep_partials=keep)
    for order in (B.cp_ring_passkv, B.cp_ring_passq):
        out, lse = order(ring)
        torch.cuda.synchronize()
        check_ring(oracle, ring, out, lse, case, keep)


def test_ring_of_more_ranks_than_one_launch_takes(oracle):
    case = ring_case(4200, [9] * 33, [5] * 33, 4, 2, 128)
    for keep in (False, True):
        ring = B.Ring(*case[0], out_dtype=torch.float32, keep_partials=keep)
        out, lse = B.cp_ring_passkv(ring)
        torch.cuda.synchronize()
        check_ring(oracle, ring, out, lse, case, keep)


# The walk behind arrival flags: uneven shards, an empty one, a rank without queries, several KV
# heads, a shard of more blocks than a workgroup lists at once, one that never arrives.
@pytest.mark.parametrize("kv_sizes,q_sizes,nh,nkv", [
    ([700, 0, 33], [520, 0, 515], 64, 4),
    ([1, 17000, 300, 0], [2048, 2050, 0, 2049], 16, 1),
])
def test_ring_walk_counts_every_key(kv_sizes, q_sizes, nh, nkv):
    n, total, t = len(kv_sizes), sum(kv_sizes), sum(q_sizes)
    ends = np.concatenate([[0], np.cumsum(kv_sizes)])
    q_pos = np.random.default_rng(t).integers(-1, total, size=t)
    rows = np.split(q_pos, np.cumsum(q_sizes)[:-1])
    args, cls = counts_case(kv_sizes, q_sizes, nh, nkv, 128, q_pos)
    for missing in (None, 0):        # shard 0 never arrives at rank 0 (its own, step 0)
        arrived = [torch.ones(n, dtype=torch.int32, device="cuda") for _ in range(n)]
        if missing is not None:
            arrived[0][0] = 0
        ring = B.Ring(*args, out_dtype=torch.float32, fused_merge=2, arrived=arrived, spin_limit=3)
        out, lse = B.cp_ring_passkv(ring)
        torch.cuda.synchronize()
        assert ring.ring_error.tolist() == [0 if missing is None else 1] + [0] * (n - 1)
        for a, r in enumerate(rows):
            if len(r) > 0:
                lo = ends[1] if a == 0 and missing is not None else 0
                check_counts(out[a], lse[a], r, cls, 128, lo)


# 33 ranks are N x N calls whose shards' position bounds are made once, in two launches (32 and 1):
# two streams, gathered queries (a call per holder, one merge), every option with keys of zero so
# that a bound of the wrong shard shows. 2050 tokens and 16 heads a rank are enough row blocks for
# two streams (no split of the KV axis), 64 are not.
@pytest.mark.parametrize("per,d", [(64, 128), (2050, 128), (40, 64)])
def test_ring_of_calls_counts_every_key(per, d):
    n = 33
    kv = [70] * 30 + [0, 145, 70]
    total = sum(kv)
    q_pos = np.sort(np.random.default_rng(per).integers(-1, total, size=n * per))
    for opts in (dict(), dict(aux_stream=torch.cuda.Stream()),
                 dict(aux_stream=torch.cuda.Stream(), keep_partials=True),
                 dict(keep_partials=True, gathered_q=True)):
        args, cls = counts_case(kv, [per] * n, 16, 1, d, q_pos)
        if "gathered_q" in opts:   # back to back in one buffer
            for i in (0, 3):
                whole = torch.cat(args[i])
                args[i][:] = [whole[r * per:(r + 1) * per] for r in range(n)]
        ring = B.Ring(*args, out_dtype=torch.float32, **opts)
        for order in ([B.cp_ring_passq] if "gathered_q" in opts else
                      [B.cp_ring_passkv, B.cp_ring_passq]):
            out, lse = order(ring)
            torch.cuda.synchronize()
            check_counts(torch.cat(out), torch.cat(lse), q_pos, cls, d)


# merged step by step in one slot: nothing behind the slot is written
def test_fused_ring_of_more_ranks_than_one_launch_takes(oracle):
    case = ring_case(4200, [9] * 33, [5] * 32 + [0], 4, 2, 128)
    ring = B.Ring(*case[0], out_dtype=torch.float32, fused_merge=True)
    block = torch.full((33, *ring.partial_out.shape[1:]), 7.0, device="cuda")
    rows = torch.full((33, *ring.partial_lse.shape[1:]), 7.0, device="cuda")
    ring.desc.partial_out, ring.desc.partial_lse = block.data_ptr(), rows.data_ptr()
    for order in (B.cp_ring_passkv, B.cp_ring_passq):
        out, lse = order(ring)
        torch.cuda.synchronize()
        check_ring(oracle, ring, out, lse, case, False)
        assert (block[1:] == 7.0).all() and (rows[1:] == 7.0).all()


# row blocks of 4 tokens: 255 and 256 of them in one call (planned; a workgroup each without a
# plan), 1024 and 1026 units of two shards kept apart (planned; not)
@pytest.mark.parametrize("shards,tokens", [(1, 1020), (1, 1021), (2, 2048), (2, 2049)])
def test_unit_limits(oracle, shards, tokens):
    nh, tkv = 64, 70
    rng = np.random.default_rng(tokens)
    q, q64 = randn(4301, (tokens, nh, 128))
    k, k64 = randn(4302, (tkv, 1, 128))
    v, v64 = randn(4303, (tkv, 1, 128))
    qp = rng.integers(-1, tkv, size=tokens)
    some = np.r_[0:5, tokens // 2 - 3:tokens // 2 + 3, tokens - 5:tokens]
    ref_o, ref_l = oracle.attn(q64[some], k64, v64, qp[some], np.arange(tkv))
    if shards == 1:
        o, l = B.cp_attn_partial(dev(q), dev(k), dev(v), i32(qp), i32(np.arange(tkv)))
    else:
        half, cut = tokens // 2, 37
        ring = B.Ring([dev(q[:half]), dev(q[half:])], [dev(k[:cut]), dev(k[cut:])],
                      [dev(v[:cut]), dev(v[cut:])], [i32(qp[:half]), i32(qp[half:])],
                      [i32(np.arange(cut)), i32(np.arange(cut, tkv))], out_dtype=torch.float32,
                      keep_partials=True)
        out, lse = B.cp_ring_passkv(ring)
        o, l = torch.cat(out), torch.cat(lse)
    torch.cuda.synchronize()
    check(o[some], l[some], ref_o, ref_l, what="sampled rows")


# fp32: 16 and 32 rows a workgroup (head_dim 64, 16384 rows), head_dim 128, lists of more than
# 256 blocks of 16 keys
@pytest.mark.parametrize("kv_sizes,q_sizes,nh,nkv,d", [
    ([17, 1], [16, 17], 4, 1, 64),
    ([300, 0, 213], [100, 0, 90], 8, 2, 64),
    ([1000, 1049], [1024, 1024], 8, 1, 64),
    ([1000, 1050], [1025, 1024], 8, 1, 64),
    ([4100, 37], [21, 12], 4, 2, 128),
])
@pytest.mark.parametrize("keep", [False, True])
def test_fp32_ring(oracle, kv_sizes, q_sizes, nh, nkv, d, keep):
    case = ring_case(4400, kv_sizes, q_sizes, nh, nkv, d, "fp32")
    ring = B.Ring(*case[0], keep_partials=keep)
    out, lse = B.cp_ring_passkv(ring)
    torch.cuda.synchronize()
    check_ring(oracle, ring, out, lse, case, keep, O_ATOL_FP32, LSE_RTOL_FP32)


# fp32: workgroups of 16 rows on either side of 512, 768 and 1024 (head_dim 64), lists of more than 512
# blocks of 16 keys, the last of them of one key; then the forms of fp32_form and the sizes on either side
# of their rules: 16 rows by 8 (256 workgroups; up to 512 of a whole prefill, and on more than 512 keys),
# 32 by 8 and by 4 (keys 257 and 256), head_dim 128 by 4 and by 8 (128 and 129 keys; 256 and 257 of more
# than 256 workgroups)
@pytest.mark.parametrize("kv_sizes,q_sizes,nh,nkv,d", [
    ([70, 59], [1000, 1048], 4, 1, 64),
    ([70, 59], [1000, 1049], 4, 1, 64),
    ([33, 300], [1536, 1536], 4, 1, 64),
    ([33, 300], [1536, 1537], 4, 1, 64),
    ([1, 64], [2048, 2048], 4, 1, 64),
    ([1, 64], [2049, 2048], 4, 1, 64),
    ([8193, 8209], [5, 3], 4, 1, 64),
    ([8193, 40], [5, 3], 4, 1, 128),
    ([15, 16, 17], [0, 1, 9], 8, 2, 128),
    ([70, 59], [400, 624], 4, 1, 64),
    ([70, 58], [400, 624], 4, 1, 64),
    ([300, 320], [310, 310], 8, 2, 64),
    ([300, 213], [600, 501], 4, 1, 64),
    ([300, 212], [600, 501], 4, 1, 64),
    ([200, 57], [1700, 1600], 4, 1, 64),
    ([200, 56], [1700, 1601], 4, 1, 64),
    ([64, 64], [5, 30], 4, 1, 128),
    ([64, 65], [5, 30], 4, 1, 128),
    ([200, 56], [500, 528], 4, 1, 128),
    ([200, 57], [500, 528], 4, 1, 128),
])
@pytest.mark.parametrize("keep", [False, True])
def test_fp32_ring_of_eight_wavefronts(oracle, kv_sizes, q_sizes, nh, nkv, d, keep):
    case = ring_case(4450, kv_sizes, q_sizes, nh, nkv, d, "fp32")
    ring = B.Ring(*case[0], keep_partials=keep)
    out, lse = B.cp_ring_passkv(ring)
    torch.cuda.synchronize()
    check_ring(oracle, ring, out, lse, case, keep, O_ATOL_FP32, LSE_RTOL_FP32)


# positions encoded in one launch (a workgroup per 1024 tokens) and in two: (sequences - 5) * lists on
# either side of 48 for 1, 2, 8 and 32 ranks, 65536 tokens and more, sequences that are empty on every
# rank, padding on both sides; many sequences over many ranks
@pytest.mark.parametrize("n,batch,length", [
    (1, 1, 1), (1, 2, 512), (3, 5, 700), (2, 63, 9), (2, 64, 9), (2, 65, 9), (17, 64, 34),
    (1, 2, 16384), (1, 2, 16385),
    (1, 29, 40), (1, 30, 40), (2, 17, 130), (2, 18, 130), (8, 8, 90), (8, 9, 90), (32, 5, 70),
    (32, 6, 70),
])
def test_packed_positions_in_one_launch(oracle, n, batch, length):
    nh, rng = 2, np.random.default_rng(4500 + batch)
    lens = np.maximum(length - np.arange(batch) % 3 * (length // 3), 0)
    if batch == 2 and length >= 16384:
        lens[:] = length            # on either side of 65536 tokens
    elif batch > 2:
        lens[1] = 0
    qs, ks, vs, ps, pk, cus = [], [], [], [], [], []
    for r in range(n):
        pos = [B.cp_shard_positions(int(x), n, r) for x in lens]
        cu = np.concatenate([[0], np.cumsum([len(p) for p in pos])]).astype(np.int32)
        p = np.concatenate(pos).astype(np.int32)
        kp, qp = p.copy(), p.copy()
        kp[rng.random(len(p)) < 0.05] = B.CP_POS_PAD_KV
        qp[rng.random(len(p)) < 0.05] = B.CP_POS_PAD_Q
        for xs, h, i in ((qs, nh, 0), (ks, 1, 1), (vs, 1, 2)):
            xs.append(randn(4510 + 3 * r + i, (len(p), h, 128)))
        ps.append(qp)
        pk.append(kp)
        cus.append(cu)
    ring = B.Ring([dev(x[0]) for x in qs], [dev(x[0]) for x in ks], [dev(x[0]) for x in vs],
                  [i32(x) for x in ps], [i32(x) for x in pk], out_dtype=torch.float32,
                  cu_seqlens_q=[i32(c) for c in cus], cu_seqlens_kv=[i32(c) for c in cus])
    out, lse = B.cp_ring_passkv(ring)
    torch.cuda.synchronize()
    for b in range(batch):
        of = [slice(c[b], c[b + 1]) for c in cus]
        kp = np.concatenate([x[s] for x, s in zip(pk, of)])
        k, v = (np.concatenate([x[1][s] for x, s in zip(xs, of)]) for xs in (ks, vs))
        for r in range(n):
            rows = np.arange(of[r].start, of[r].stop)
            if len(rows) > 200:     # (the oracle is the slow side)
                rows = np.unique(np.concatenate([rows[:40], rows[-40:], rng.choice(rows, 40)]))
            if len(rows) == 0:
                continue
            ref_o, ref_l = oracle.attn(qs[r][1][rows], k, v, ps[r][rows], kp)
            at = torch.as_tensor(rows).cuda()
            check(out[r][at], lse[r][at], ref_o, ref_l, what="rank %d sequence %d" % (r, b))


# batches on either side of the 1024 sequences whose spans the encode kernel scans by itself
@pytest.mark.parametrize("batch", [1023, 1024, 1025])
def test_packed_batch_of_many_sequences(oracle, batch):
    nh = 2
    lens = 1 + np.arange(batch) % 4
    cu = np.concatenate([[0], np.cumsum(lens)])
    total = int(cu[-1])
    pos = np.concatenate([np.arange(n) for n in lens])
    q, q64 = randn(4501, (total, nh, 128))
    k, k64 = randn(4502, (total, 1, 128))
    v, v64 = randn(4503, (total, 1, 128))
    o, l = B.cp_attn_partial(dev(q), dev(k), dev(v), i32(pos), i32(pos), i32(cu), i32(cu))
    torch.cuda.synchronize()
    ref_o, ref_l = oracle.attn(q64, k64, v64, pos, pos, cu, cu)
    check(o, l, ref_o, ref_l, what="batch %d" % batch)


# flat decode over several holders: ranges of 64 keys (the smallest) with a short last one, more
# holders than fit one round of workgroups per KV head, sequences that end at a range's end, in
# its last key, or hold nothing on a holder
@pytest.mark.parametrize("n,lengths,nh,nkv", [
    (2, [[64, 128, 1, 63], [65, 0, 64, 128]], 16, 1),
    (3, [[700, 33], [1, 0], [0, 9000]], 8, 2),
    (33, [[5, 60]] * 33, 32, 16),
    (2, [[30000, 9, 41], [16, 31000, 17]], 16, 1),
])
def test_decode_ring_ranges(oracle, n, lengths, nh, nkv):
    batch = len(lengths[0])
    m = (batch + n - 1) // n                  # queries per rank; equal, so the batch is filled up
    lengths = [list(x) + [0] * (m * n - batch) for x in lengths]
    batch = m * n
    q, q64 = randn(4601, (batch, nh, 128))
    keys = [sum(x[b] for x in lengths) for b in range(batch)]
    ks, vs, kps, cus, refs = [], [], [], [], [([], [], []) for _ in range(batch)]
    begin = [0] * batch
    for r, ls in enumerate(lengths):
        total = sum(ls)
        k, k64 = randn(4610 + 2 * r, (total, nkv, 128))
        v, v64 = randn(4611 + 2 * r, (total, nkv, 128))
        cu = np.concatenate([[0], np.cumsum(ls)])
        pos = []
        for b, L in enumerate(ls):
            p = begin[b] + np.arange(L)
            begin[b] += L
            pos.append(p)
            for dst, src in zip(refs[b], (k64[cu[b]:cu[b + 1]], v64[cu[b]:cu[b + 1]], p)):
                dst.append(src)
        ks.append(dev(k)); vs.append(dev(v)); cus.append(i32(cu)); kps.append(i32(np.concatenate(pos)))
    bid = np.random.default_rng(46).permutation(batch)
    qp = np.array([max(0, keys[b] - 1 - (b % 3)) for b in bid])   # (some keys lie behind the query)
    qd, qpd, bd = dev(q), i32(qp), i32(bid)
    sl = [slice(r * m, (r + 1) * m) for r in range(n)]
    ring = B.Ring([qd[x] for x in sl], ks, vs, [qpd[x] for x in sl], kps, out_dtype=torch.float32,
                  keep_partials=True, gathered_q=True, cu_seqlens_kv=cus, bid=[bd[x] for x in sl],
                  unique_bid=True)
    out, lse = B.cp_ring_passq_decode(ring)
    torch.cuda.synchronize()
    for i, b in enumerate(bid):
        k64, v64, p = (np.concatenate(x) for x in refs[b])
        if len(p) == 0:
            ref_o, ref_l = np.zeros((1, nh, 128)), np.full((1, nh), -np.inf)
        else:
            ref_o, ref_l = oracle.attn(q64[i:i + 1], k64, v64, qp[i:i + 1], p)
        check(ring.out_all[i:i + 1], ring.lse_all[i:i + 1], ref_o, ref_l, what="sequence %d" % b)


# bf16 inputs of head_dim 64: the probabilities keep their 24 bits, so that what separates an fp32
# result from the exact one is fp32 sums over the keys. A sum of n terms in fp32 errs by about
# 2^-24 sqrt(n) of its size; probabilities rounded to bf16 would err by 1e-3 whatever n.
@pytest.mark.parametrize("kv_sizes,q_sizes,nh,nkv", [
    ([300], [300], 8, 8),            # a workgroup per unit
    ([769, 331], [140, 57], 16, 2),  # equal shares
    ([420], [1040], 64, 1),          # more row blocks than CUs
])
def test_head_dim_64_keeps_fp32_probabilities(oracle, kv_sizes, q_sizes, nh, nkv):
    case = ring_case(4700, kv_sizes, q_sizes, nh, nkv, 64)
    out, _ = B.cp_ring_passkv(B.Ring(*case[0], out_dtype=torch.float32))
    torch.cuda.synchronize()
    _, rows, _, q_all, (q64, k64, v64) = case
    ref_o, _ = oracle.attn(q64, k64, v64, q_all, np.arange(len(k64)))
    err = rel_l2(torch.cat(out), np.concatenate([ref_o[r] for r in rows]))
    assert err < 2.0 ** -24 * np.sqrt(sum(kv_sizes)), err


# a position below zero that is not the padding's is a position like any other
def test_head_dim_64_takes_negative_positions(oracle):
    q, q64 = randn(4711, (40, 4, 64))
    k, k64 = randn(4712, (90, 1, 64))
    v, v64 = randn(4713, (90, 1, 64))
    qp, kp = np.arange(40) - 30, np.arange(90) - 50
    qp[qp == B.CP_POS_PAD_Q] = 5
    o, l = B.cp_attn_partial(dev(q), dev(k), dev(v), i32(qp), i32(kp), out_dtype=torch.float32)
    torch.cuda.synchronize()
    check(o, l, *oracle.attn(q64, k64, v64, qp, kp))


# The merge of a flat decode call: 256 and 257 parts of 64 keys, all 512 ranges, one part; 160 and 176
# rows (four workgroups a row and one); 63, 64 and 65 sequences (whose boundaries fit a wavefront or not).
@pytest.mark.parametrize("lengths,nh,nkv", [
    ([16384], 16, 1), ([16385], 16, 1), ([130001], 3, 1), ([5, 1, 64, 63, 65], 16, 1),
    ([700, 3000, 20, 64, 128, 900, 1, 333, 2000, 77], 16, 1),
    ([700, 3000, 20, 64, 128, 900, 1, 333, 2000, 77, 5000], 16, 1),
    ([9000, 8000], 8, 4), (list(range(1, 64)), 2, 1), (list(range(64, 0, -1)), 2, 1),
    (list(range(3, 68)), 2, 2),
])
def test_flat_decode_merge_counts_every_key(lengths, nh, nkv):
    batch, cu = len(lengths), np.concatenate([[0], np.cumsum(lengths)])
    q, _ = randn(61, (batch, nh, 128))
    k = torch.zeros((int(cu[-1]), nkv, 128), dtype=torch.bfloat16, device="cuda")
    v = torch.zeros_like(k)
    pos = np.concatenate([np.arange(n) for n in lengths])
    cls = (pos // 16 + pos) % 128
    v[torch.arange(len(pos)), :, torch.as_tensor(cls)] = 1.0
    bid = np.random.default_rng(batch).permutation(batch)
    q_pos = np.array([lengths[b] - 1 - (b % 3 == 2) * (lengths[b] // 2) for b in bid])
    for dtype in (torch.float32, torch.bfloat16):
        o, l = B.cp_attn_decode(dev(q), k, v, i32(q_pos), i32(pos), i32(cu), i32(bid),
                                out_dtype=dtype, unique_bid=True)
        torch.cuda.synchronize()
        if dtype == torch.bfloat16:   # (rounded once)
            assert torch.equal(o, whole.to(torch.bfloat16))
            continue
        whole = o
        for i, b in enumerate(bid):
            check_counts(o[i:i + 1], l[i:i + 1], q_pos[i:i + 1], cls[cu[b]:cu[b + 1]], 128)


# The flat decode kernel holds a probability to 16 bits (two bf16 terms) or better: each errs by up
# to 2^-17 of itself, independently, and the fp32 sums by 2^-24 sqrt(keys); with one term it would be
# 2^-9. (Error of a whole result, of which the probabilities' is the root mean square: below 2^-17.)
def test_flat_decode_keeps_probabilities_to_16_bits(oracle):
    lens, nh = [40, 3000, 700], 16
    cu = np.concatenate([[0], np.cumsum(lens)])
    q, q64 = randn(4801, (3, nh, 128))
    k, k64 = randn(4802, (sum(lens), 1, 128))
    v, v64 = randn(4803, (sum(lens), 1, 128))
    pos = np.concatenate([np.arange(n) for n in lens])
    o, _ = B.cp_attn_decode(dev(q), dev(k), dev(v), i32(np.array(lens) - 1), i32(pos), i32(cu),
                            i32(np.arange(3)), out_dtype=torch.float32, unique_bid=True)
    torch.cuda.synchronize()
    ref = np.concatenate([oracle.attn(q64[b:b + 1], k64[cu[b]:cu[b + 1]], v64[cu[b]:cu[b + 1]],
                                      np.array([n - 1]), np.arange(n))[0]
                          for b, n in enumerate(lens)])
    err = rel_l2(o, ref)
    assert err < 2.0 ** -17, err
