"""The launch rules of csrc/cp_launch_rules.h, compiled for the host and checked over ranges of sizes
that a few calls on a GPU cannot cover. No GPU needed."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2411_01783_amd", "csrc")

SHIM = r"""
#include "cp_launch_rules.h"
extern "C" {
// where the workgroups of a grid run: x + nx * z of each, in dispatch order
int placed(int parts, int row_blocks, int n_kv_heads, int nz, int n_blocks, int32_t* out) {
  const int nx = row_blocks * n_kv_heads;
  const bool slice =
      cp::xcd_slice_applies((cp::GridParts)parts, row_blocks, n_kv_heads, nz, n_blocks);
  for (int i = 0; i < nx * nz; ++i) {
    cp::GridPos at = {i % nx, i / nx};
    if (slice) at = cp::xcd_slice(at.x, at.z, nx, nz);
    out[i] = at.x < 0 || at.x >= nx || at.z < 0 || at.z >= nz ? -1 : at.x + nx * at.z;
  }
  return slice;
}
int shares_grouped(int head_dim, int units) { return cp::shares_grouped(head_dim, units); }
int shards_alike(int n, const int32_t* n_kv, int64_t total_q) {
  return cp::shards_alike(n, n_kv, total_q);
}
int encode_in_one_launch(int64_t batch, int64_t lists, int64_t tokens) {
  return cp::encode_in_one_launch(batch, lists, tokens);
}
int fp32_form(int head_dim, int64_t rows, int64_t n_kv_heads, int64_t shards, int kept_apart,
              int64_t total_q, int64_t total_keys) {
  const cp::Fp32Form f = cp::fp32_form(head_dim, rows, n_kv_heads, shards, kept_apart != 0, total_q,
                                       total_keys);
  return f.rows * 10 + f.waves;
}
// begin: of the ranks, in tokens of `group` rows; out: of the 2N + 1 chunks, in blocks of `rows` rows
// (`apart`: which do not straddle ranks)
void chunk_begins(int B, int N, const int32_t* begin, uint32_t group, uint32_t rows, int apart,
                  int32_t* out) {
  cp::ChunkRule rule = cp::chunk_rule(N, begin, group);
  if (apart) rule = cp::chunk_rule_in_blocks(N, rule, rows, B);
  for (int j = 0; j <= 2 * N; ++j) out[j] = cp::chunk_begin(j, B, N, rule, apart ? 1 : rows);
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = str(d / "rules.cpp"), str(d / "rules.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.check_call([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-Wall", "-Werror",
                           "-fPIC", "-shared", "-I", CSRC, src, "-o", lib])
    return ctypes.CDLL(lib)


VISIBLE, BY_INDEX, ALIKE, OTHER = range(4)


def placed(rules, parts, row_blocks, nkv, nz, n_blocks=1 << 20):
    out = np.empty(row_blocks * nkv * nz, dtype=np.int32)
    moved = rules.placed(parts, row_blocks, nkv, nz, n_blocks, out.ctypes.data_as(ctypes.c_void_p))
    return out, bool(moved)


def test_every_workgroup_of_a_grid_runs_once(rules):
    moves = 0
    for nz in list(range(1, 41)) + [48, 64, 69, 128]:
        for row_blocks, nkv in [(x, 1) for x in range(1, 70)] + [(2, 2), (3, 4), (5, 2), (128, 1)]:
            for parts in (VISIBLE, BY_INDEX, ALIKE, OTHER):
                out, moved = placed(rules, parts, row_blocks, nkv, nz)
                assert np.array_equal(np.sort(out), np.arange(row_blocks * nkv * nz))
                moves += moved and not np.array_equal(out, np.arange(len(out)))
    assert moves > 50


# Work per z in proportion. Workgroups go to the eight XCDs in turn, and the time is that of the busiest
# one. Shards that are not alike (a holder with more keys, contiguous ones under a causal mask) stay as
# dispatched; what is placed is the same work for every XCD.
@pytest.mark.parametrize("shares", [
    [1] * 7 + [2], [1] * 15 + [2], [3, 1], [1, 1, 1, 4], list(range(8, 0, -1)), [7, 5, 3, 1], [1, 0],
    [4] * 8 + [1] * 8, [1, 1, 0, 0], [1] * 8 + [0] * 8, [1] * 4 + [0] * 12, [5] + [1] * 31, [1] * 6,
    [1] * 16,
])
def test_no_xcd_gets_more_than_its_part(rules, shares):
    for sub in (1, 2, 3, 4, 8, 16):
        work = np.repeat(np.array(shares, dtype=np.int64), sub)
        nz = len(work)
        n_kv = (ctypes.c_int32 * len(shares))(*[8192 * x for x in shares])
        alike = rules.shards_alike(len(shares), n_kv, ctypes.c_int64(128))
        assert bool(alike) == (len(set(shares)) == 1)
        for row_blocks in (2, 4, 8, 12, 16, 32, 64, 128, 192, 256, 512):
            out, _ = placed(rules, ALIKE if alike else OTHER, row_blocks, 1, nz)
            load = [work[out[x::8] // row_blocks].sum() for x in range(8)]
            plain = [work[np.arange(x, row_blocks * nz, 8) // row_blocks].sum() for x in range(8)]
            assert max(load) <= max(plain), (row_blocks, nz)


def test_shards_of_a_prefill_are_not_alike(rules):
    n_kv = (ctypes.c_int32 * 8)(*[1000] * 8)
    assert rules.shards_alike(8, n_kv, ctypes.c_int64(1000))
    assert not rules.shards_alike(8, n_kv, ctypes.c_int64(1001))   # (contiguous, causal: very unlike)


# Parts of one shard by index, under a causal mask the first ones are the long walks: spread over the XCDs.
def test_parts_by_index_are_spread(rules):
    for row_blocks in (2, 4, 8, 16, 32, 64, 192):
        for nz in (2, 4, 8, 16, 32, 64):
            out, _ = placed(rules, BY_INDEX, row_blocks, 1, nz)
            work = np.arange(nz, 0, -1)
            load = np.array([work[out[x::8] // row_blocks].sum() for x in range(8)])
            if row_blocks * nz >= 64:
                assert load.max() <= 1.25 * load.mean(), (row_blocks, nz)


# and what the placement is for: a z on as few XCDs as can be
@pytest.mark.parametrize("parts,row_blocks,nkv,nz,xcds", [
    (ALIKE, 8, 1, 32, 1), (ALIKE, 4, 2, 30, 4), (VISIBLE, 12, 1, 20, 2), (VISIBLE, 2, 2, 64, 1),
    (BY_INDEX, 8, 1, 32, 1),
])
def test_workgroups_on_the_same_keys_share_xcds(rules, parts, row_blocks, nkv, nz, xcds):
    out, moved = placed(rules, parts, row_blocks, nkv, nz, 4096)
    assert moved
    for z in range(nz):
        assert len(set(np.flatnonzero(out // (row_blocks * nkv) == z) % 8)) == xcds


# head_dim, units, time with neighbouring shares on one XCD over that as dispatched (16384 to 29000 keys)
@pytest.mark.parametrize("d,units,ratio", [
    (128, 8, 1.03), (128, 12, 1.035), (128, 20, 1.03), (128, 24, 1.02), (128, 28, .97), (128, 64, .965),
    (128, 320, .95), (64, 16, .97), (64, 48, .96),
])
def test_shares_of_few_units_are_not_grouped(rules, d, units, ratio):
    assert bool(rules.shares_grouped(d, units)) == (ratio < 1)


# Ranks, sequences, and the time of a whole packed call with its positions encoded in one launch over
# that in two (prompts of 64 or 256 tokens, MI355X): whatever loses 2 % or more takes two, whatever
# gains 4 % or more takes one. (In one launch a wavefront walks sequences * ranks / 8 pieces one by one.)
@pytest.mark.parametrize("ranks,batch,ratio", [
    (1, 1, .89), (1, 8, .88), (1, 16, .92), (1, 24, .96), (1, 40, 1.03), (1, 64, 1.12),
    (2, 6, .92), (2, 12, .96), (2, 24, 1.04), (3, 8, .96), (4, 2, .87), (4, 8, .96), (4, 14, 1.02),
    (4, 32, 1.21), (4, 64, 1.54), (8, 2, .87), (8, 5, .96), (16, 1, .84), (16, 4, .96), (16, 8, 1.07),
    (16, 16, 1.31), (16, 64, 2.59), (32, 1, .84), (32, 5, .96), (32, 8, 1.12), (32, 64, 3.23),
])
def test_positions_of_many_pieces_take_two_launches(rules, ranks, batch, ratio):
    one = rules.encode_in_one_launch
    one.argtypes = [ctypes.c_int64] * 3
    assert ratio >= 1.02 or ratio <= 0.96
    assert bool(one(batch, 2 * ranks, batch * 128)) == (ratio < 1)
    assert not one(1, 2 * ranks, 65537)


def test_pieces_of_one_launch_fit_a_wavefront(rules):
    one = rules.encode_in_one_launch
    one.argtypes = [ctypes.c_int64] * 3
    for lists in range(2, 65):       # kMaxTable ranks and shards
        for batch in range(1, 2000):
            if one(batch, lists, 1):   # a lane per sequence, a lane per piece of 16 wavefronts
                assert batch <= 64 and -(-batch * lists // 16) <= 64


def shards(total, N):
    """Lengths of the early and late chunks of N ranks, as cp_shard_positions deals them."""
    size = -(-total // (2 * N))
    length = lambda c: min((c + 1) * size, total) - min(c * size, total)
    return np.array([[length(r), length(2 * N - 1 - r)] for r in range(N)])


def chunk_begins(rules, B, sizes, group, rows, apart=False):
    N = len(sizes)
    at = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    begin = np.empty(2 * N + 1, np.int32)
    rules.chunk_begins(B, N, at.ctypes.data_as(ctypes.c_void_p), ctypes.c_uint32(group),
                       ctypes.c_uint32(rows), int(apart), begin.ctypes.data_as(ctypes.c_void_p))
    assert begin[0] == 0 and begin[-1] == B and np.all(np.diff(begin) >= 0), (sizes, group, rows)
    return begin


def dispatch_order(rules, B, sizes, group, rows, apart=False):
    """Row blocks as ordered_row_block hands them out: the late chunks of ranks 0, 1, .., then the
    early ones of ranks N - 1, .., 0, each from its end."""
    N, begin = len(sizes), chunk_begins(rules, B, sizes, group, rows, apart)
    chunks = [2 * r + 1 for r in range(N)] + [2 * r for r in reversed(range(N))]
    return np.concatenate([np.arange(begin[j], begin[j + 1])[::-1] for j in chunks])


# Row blocks of the fp32 kernel (16 and 32 rows) and of the bf16 kernel, over chunks of any length: equal
# ones and, where the total is no multiple of 2N, short and empty ones at the end of the sequence.
@pytest.mark.parametrize("rows", [16, 32, 256])
@pytest.mark.parametrize("group", [1, 4, 16])
def test_row_blocks_with_late_rows_go_first(rules, rows, group):
    rng = np.random.default_rng(rows + group)
    for N in (2, 3, 4, 7, 8, 16, 32):
        chunks = list(range(3, 60, 7)) + [128, 165, 225, 256, 450, 1000, 1042, 2079, 3117]
        totals = [2 * N * c - k for c in chunks for k in {0, 1, N, 2 * N - 1, int(rng.integers(2 * N))}]
        for total in totals:
            parts = shards(total, N)
            B = -(-total * group // rows)
            order = dispatch_order(rules, B, parts.sum(1), group, rows)
            assert np.array_equal(np.sort(order), np.arange(B))
            late = np.repeat(np.tile([False, True], N), parts.ravel() * group)
            has_late = np.logical_or.reduceat(late, np.arange(B) * rows)
            # (where a late chunk is empty, a block of two ranks' early rows may be among the late ones)
            empty = int((parts[:, 1] == 0).sum())
            assert np.flatnonzero(has_late[order]).max(initial=-1) < has_late.sum() + empty, (N, total)


# The walk behind flags, whose row blocks do not straddle ranks. (Short late chunks are taken for whole
# ones but for what the row blocks are fewer: a boundary can be a block off where they are several.)
@pytest.mark.parametrize("group", [1, 4, 16])
def test_row_blocks_of_whole_ranks_go_late_chunk_first(rules, group):
    rng, rows = np.random.default_rng(group), 256
    for N in (2, 4, 8, 16, 32):
        for chunk in [128, 165, 256, 450, 1000, 1042, 2079, 2431, 3117]:
            for k in {0, 1, N, 2 * N - 1, int(rng.integers(2 * N))}:
                parts = shards(2 * N * chunk - k, N)
                per = -(-parts.sum(1) * group // rows)
                order = dispatch_order(rules, int(per.sum()), parts.sum(1), group, rows, True)
                assert np.array_equal(np.sort(order), np.arange(per.sum()))
                # (the first block with a late row of every rank)
                begin = np.concatenate([[0], np.cumsum(per)])
                late = np.zeros(per.sum(), bool)
                for r in range(N):
                    if parts[r, 1] > 0:
                        late[begin[r] + parts[r, 0] * group // rows:begin[r + 1]] = True
                # (a block a rank where a late chunk ends a block early or has no row)
                short = int((per < per.max()).sum() + (parts[:, 1] == 0).sum())
                assert np.flatnonzero(late[order]).max() < late.sum() + short, (N, chunk, k)


def test_row_blocks_are_all_handed_out(rules):
    rng = np.random.default_rng(5)
    for N in range(2, 33):
        for total in list(range(1, 200)) + [4095, 65537]:
            sizes = rng.multinomial(total, rng.dirichlet(np.full(N, .3)))
            for group, rows in ((1, 16), (3, 32), (16, 256)):
                B = -(-total * group // rows)
                assert np.array_equal(np.sort(dispatch_order(rules, B, sizes, group, rows)), np.arange(B))
    # as many rows as are accepted, dealt evenly and to one rank: boundaries only, within 32 bits
    for N in (2, 3, 32):
        for sizes in ([0x7fffffff // N] * N, [0x7fffffff] + [0] * (N - 1), [0] * (N - 1) + [0x7fffffff]):
            chunk_begins(rules, -(-sum(sizes) // 16), sizes, 1, 16)
            chunk_begins(rules, sum(-(-n // 16) for n in sizes), sizes, 1, 16, True)


# Calls of the fp32 kernel whose time with another form of workgroup (rows, wavefronts) was measured:
# head_dim, queries, heads, KV heads, shards, kept apart, keys; the form that has to be taken, and one that
# loses to it by 4 % or more (us of both, MI355X).
FP32_FORMS = [
    (64, 512, 4, 1, 1, 0, 16, (16, 4), (16, 8), 6.0, 6.6),
    (64, 2048, 4, 1, 1, 0, 16, (16, 4), (16, 8), 6.8, 11.1),
    (64, 2048, 4, 1, 1, 0, 512, (16, 4), (16, 8), 21.5, 25.5),
    (64, 1024, 8, 2, 1, 0, 256, (16, 4), (16, 8), 13.9, 18.5),
    (64, 512, 4, 1, 4, 1, 2048, (16, 4), (16, 8), 26.4, 30.9),
    (64, 1024, 4, 1, 2, 1, 1024, (16, 4), (16, 8), 25.6, 26.8),
    (64, 512, 8, 1, 2, 1, 512, (16, 4), (16, 8), 18.4, 22.3),
    (64, 512, 4, 1, 1, 0, 512, (16, 8), (16, 4), 13.6, 17.2),
    (64, 512, 4, 1, 2, 0, 512, (16, 8), (16, 4), 14.2, 17.5),
    (64, 1320, 4, 1, 4, 0, 1320, (16, 8), (16, 4), 25.4, 37.0),
    (64, 2048, 4, 1, 2, 0, 2048, (16, 8), (16, 4), 43.0, 54.3),
    (64, 540, 8, 2, 1, 0, 540, (16, 8), (16, 4), 14.1, 19.0),
    (64, 1500, 4, 1, 1, 0, 3000, (16, 8), (16, 4), 67.4, 77.7),
    (64, 3040, 4, 1, 2, 0, 3040, (16, 4), (16, 8), 80.2, 89.0),
    (64, 4096, 4, 1, 1, 0, 16, (32, 4), (16, 4), 9.4, 11.2),
    (64, 4096, 4, 1, 1, 0, 256, (32, 4), (32, 8), 20.3, 27.3),
    (64, 512, 4, 1, 8, 1, 512, (32, 4), (32, 8), 17.2, 25.1),
    (64, 1024, 4, 1, 4, 1, 1024, (32, 4), (32, 8), 26.0, 30.3),
    (64, 3600, 4, 1, 2, 0, 3600, (32, 8), (16, 4), 93.0, 112.7),
    (64, 2048, 4, 1, 2, 1, 2048, (32, 8), (32, 4), 55.4, 60.3),
    (64, 5000, 4, 1, 2, 0, 5000, (32, 4), (32, 8), 202.7, 224.1),
    (64, 2048, 4, 1, 8, 1, 512, (16, 4), (32, 8), 64.0, 86.4),
    (128, 512, 4, 1, 1, 0, 64, (16, 4), (16, 8), 7.5, 8.6),
    (128, 2048, 4, 1, 8, 1, 512, (16, 4), (16, 8), 83.6, 136.8),
    (128, 2048, 8, 1, 8, 1, 2048, (16, 4), (16, 8), 233.5, 357.0),
    (128, 2048, 4, 1, 1, 0, 256, (16, 4), (16, 8), 22.2, 27.7),
    (128, 512, 4, 1, 1, 0, 512, (16, 8), (16, 4), 20.6, 25.2),
    (128, 1100, 4, 1, 2, 0, 1100, (16, 8), (16, 4), 35.8, 51.2),
    (128, 512, 8, 2, 1, 0, 2048, (16, 8), (16, 4), 60.5, 84.1),
]


@pytest.mark.parametrize("case", FP32_FORMS)
def test_fp32_workgroups_are_of_the_form_that_was_faster(rules, case):
    d, q, nh, nkv, shards, apart, keys, form, other, us, us_other = case
    assert us_other >= 1.04 * us and other != form
    f = rules.fp32_form
    f.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int] + [ctypes.c_int64] * 2
    rows, waves = divmod(f(d, q * (nh // nkv), nkv, shards, apart, q, keys), 10)
    assert (rows, waves) == form
