"""GPU parity: specexit_verify_attn against the oracle."""
import numpy as np
import pytest
import torch

from workloads import gen

import harness as H
from harness import TOL, gpu_verify_attn, oracle_verify_attn, rel_err

pytestmark = pytest.mark.gpu


def case(shape, seed, tree=False, paged=None):
    L = gen.context_lengths(shape, seed)
    kv = gen.kv_cache(shape, L, shape.n_q, seed, paged=paged)
    q = gen.queries(shape, seed)
    mask = None
    if tree:
        mask = gen.ancestor_masks(gen.random_tree_parents(shape, seed))
    return L, kv, q, mask


def check(shape, L, kv, q, mask, only=None, label=""):
    print(f"verify_attn {label}: dtype={shape.dtype} B={shape.B} n_q={shape.n_q} Hq={shape.Hq} Hkv={shape.Hkv} "
          f"d={shape.d} L={L.tolist()[:8]} paged={kv.paged} tree={mask is not None}", flush=True)
    got = gpu_verify_attn(shape, kv, q, L, mask)
    ref = oracle_verify_attn(kv, q, L, mask, only=only)
    if only is not None:
        sel = tuple(np.array(only).T)
        got, ref = got[sel], ref[sel]
    assert np.isfinite(got).all()
    err = rel_err(got, ref)
    assert err < TOL[shape.dtype], err
    return err


def test_tiny_fp32_config():
    shape = gen.config(0)
    L, kv, q, mask = case(shape, 0)
    check(shape, L, kv, q, mask, label="config 0")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
def test_small_chain_ragged_lengths(dtype, d):
    shape = gen.scaled(gen.config(1), dtype=dtype, B=5, Hq=8, Hkv=2, d=d, n_q=7, ctx=(0, 700))
    L, kv, q, mask = case(shape, 1)
    L[0] = 0                       # empty context: only the block itself is visible
    L[1] = 121                     # not a multiple of any tile
    check(shape, L, kv, q, mask, label="chain ragged")


@pytest.mark.parametrize("paged", [False, True])
def test_small_tree(paged):
    shape = gen.scaled(gen.config(3), B=3, Hq=8, Hkv=2, ctx=(100, 900))
    L, kv, q, mask = case(shape, 2, tree=True, paged=paged)
    check(shape, L, kv, q, mask, label="tree")


@pytest.mark.parametrize("dtype,B,paged", [("bf16", 1024, False), ("bf16", 333, True), ("f32", 1024, False)])
def test_many_short_sequences(dtype, B, paged):
    # the most sequences a launch takes (the length table spans sixteen 64-lane rounds) and an odd
    # count: every workgroup's share of the keys crosses several (sequence, KV head) units, some empty
    shape = gen.scaled(gen.config(2), dtype=dtype, B=B, Hq=4, Hkv=2, n_q=2, ctx=(0, 150))
    L, kv, q, mask = case(shape, 7, paged=paged)
    L[0] = 0
    L[B - 1] = 150
    check(shape, L, kv, q, mask, label="many sequences")


@pytest.mark.parametrize("n_q,Hq,Hkv,page", [(1, 4, 1, 16), (4, 8, 2, 16), (5, 8, 2, 32), (16, 8, 2, 0), (16, 8, 2, 64), (9, 16, 2, 128),
                                             (24, 4, 1, 16), (32, 4, 1, 32), (32, 4, 1, 0)])
def test_narrow_heads_at_tile_edges(n_q, Hq, Hkv, page):
    # 64-wide heads on the matrix cores: one to eight row tiles with and without a ragged last one, pages
    # below, at and above the 32-key tile, lengths around the tile and granule edges.  Probabilities keep
    # 16 bits of mantissa, so the error is the bf16 rounding of the output: at most 2^-9 of the largest value.
    shape = gen.scaled(gen.config(1), B=6, Hq=Hq, Hkv=Hkv, d=64, n_q=n_q, k=min(5, max(n_q - 1, 1)), ctx=(0, 900), page_size=page or 16)
    L, kv, q, mask = case(shape, 11, tree=n_q > 1 and page != 0, paged=page > 0)
    for b, n in enumerate((0, 31, 32, 64 - n_q if n_q < 64 else 1, 63)):
        L[b] = n
    err = check(shape, L, kv, q, mask, label=f"d64 page {page}")
    assert err < 2.0 ** -8


@pytest.mark.parametrize("B,n_q,page,d", [(2, 5, 16, 64), (2, 16, 0, 64), (40, 3, 64, 64), (40, 7, 64, 64), (2, 5, 16, 128), (2, 12, 0, 128), (40, 3, 64, 128), (40, 7, 64, 128)])
def test_infinite_values_of_narrow_heads(B, n_q, page, d):
    # 64-wide heads, and 128-wide ones of up to 48 rows per KV head: an infinite V entry that a row sees makes its column of
    # that row infinite, with its sign (the probability is positive), and changes no other column.  The last case of either width has
    # the rows (2240 x 80 units on 320 workgroups) that a wave each merges, the others a workgroup each.
    shape = gen.scaled(gen.config(1), B=B, Hq=8, Hkv=2, d=d, n_q=n_q, ctx=(20, 500), page_size=page or 16)
    L, kv, q, _ = case(shape, 5, paged=page > 0)
    # (sequence, KV head, entry, column, value); the last one is the block's last entry, which only the last query sees
    put = [(0, 0, 3, 5, np.inf), (0, 1, int(L[0]) - 1, 63, -np.inf), (1, 0, 17, 0, -np.inf), (1, 0, 19, 0, -np.inf), (1, 1, int(L[1]) + n_q - 1, 8, np.inf)]
    for b, g, p, c, x in put:
        if kv.paged:
            kv.v[kv.page_table[b, p // kv.page_size], g, p % kv.page_size, c] = x
        else:
            kv.v[b, g, p, c] = x
    print(f"infinite V: B={B} n_q={n_q} page={page}", flush=True)
    got = gpu_verify_attn(shape, kv, q, L, None)
    with np.errstate(invalid="ignore"):
        ref = oracle_verify_attn(kv, q, L, None)
    plain = np.ones(got.shape, bool)
    G = shape.Hq // shape.Hkv
    for b, g, p, c, x in put:
        rows = slice(n_q - 1, None) if p >= L[b] else slice(None)
        assert (got[b, rows, g * G:(g + 1) * G, c] == x).all(), (b, g, p, c, got[b, rows, g * G:(g + 1) * G, c])
        plain[b, :, g * G:(g + 1) * G, c] = False
    assert np.isfinite(got[plain]).all()
    assert rel_err(got[plain], ref[plain]) < TOL["bf16"]


@pytest.mark.parametrize("d,n_q,every", [(128, 16, 4), (128, 7, 4), (64, 7, 4), (128, 16, 1), (64, 7, 1)])
def test_scores_that_are_nan_are_not_passed_over(d, n_q, every):
    # keys with a NaN, at least one for each lane that a row's scores lie in, in the first of several segments: its maximum then knows
    # no number, and its weight must not become 0.  Every query sees these keys, so all rows of their KV head are NaN.
    shape = gen.scaled(gen.config(1), B=2, Hq=8, Hkv=2, d=d, n_q=n_q, k=n_q - 1, ctx=(300, 300))
    L, kv, q, _ = case(shape, 8, paged=False)
    kv.k[1, 0, 0:64:every, 3] = np.nan
    got = gpu_verify_attn(shape, kv, q, L, None)
    assert np.isnan(got[1, :, :4]).all()
    assert np.isfinite(got[1, :, 4:]).all() and np.isfinite(got[0]).all()


@pytest.mark.parametrize("n_q,L,paged", [(4, (3000,), False), (7, (4096,), False), (12, (900, 2500), True), (7, (700, 1500, 400, 1100, 900, 300), True)])
def test_probabilities_of_few_wide_rows_have_two_parts(n_q, L, paged):
    # 128-wide heads of up to 48 rows per KV head: what is left of the error is the rounding of the output to bf16, 2^-9 / sqrt(3) of a
    # value at most, three quarters of that on average over a power of two's range.  Probabilities of 8 bits add 0.6 times as much
    # again, squared (2.05e-3 for 1.65e-3).
    shape = gen.scaled(gen.config(1), B=len(L), Hq=8, Hkv=2, d=128, n_q=n_q, k=max(n_q - 1, 1), ctx=(0, 1))
    L = np.array(L, np.int32)
    kv, q = gen.kv_cache(shape, L, n_q, 21, paged=paged), gen.queries(shape, 21)
    got = gpu_verify_attn(shape, kv, q, L, None)
    ref = oracle_verify_attn(kv, q, L, None)
    rounding = np.linalg.norm(gen.round_to_bf16(ref.astype(np.float32)) - ref) / np.linalg.norm(ref)
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print(f"  {n_q} queries, {L.tolist()}: {err:.3e}, of that the output's rounding {rounding:.3e}", flush=True)
    assert err < 1.05 * rounding


@pytest.mark.parametrize("dtype,d,n_q,B,long", [("bf16", 64, 3, 70, 9000), ("bf16", 128, 3, 70, 9000), ("f32", 64, 3, 70, 9000), ("bf16", 64, 5, 70, 9000),
                                               ("bf16", 128, 5, 70, 9000), ("bf16", 128, 3, 50, 20000), ("bf16", 128, 9, 40, 9000), ("f32", 128, 3, 50, 20000)])
def test_one_long_sequence_among_short_ones(dtype, d, n_q, B, long):
    # one unit with more segments than a wave has lanes among many of one or two.  Merged by a wave per output row from 256 rows per segment
    # of an average unit on: rows x units above 256 times the launch's workgroups, which are 256 for fp32 and for 128-wide heads of up to
    # 16 rows per KV head, 512 else.  So a workgroup per row has the 64-wide heads of three queries (840 x 140 against 256 x 512) and the
    # 128-wide ones of fifty and forty sequences (600 x 100 against 256 x 256; 1440 x 80 of 18 rows per KV head against 256 x 512).
    shape = gen.scaled(gen.config(1), dtype=dtype, B=B, Hq=4, Hkv=2, d=d, n_q=n_q, ctx=(0, 40))
    L = gen.context_lengths(shape, 3)
    L[33] = long
    kv = gen.kv_cache(shape, L, shape.n_q, 3, paged=True)
    check(shape, L, kv, gen.queries(shape, 3), None, label="one long sequence")


@pytest.mark.parametrize("d,n_q,L,page", [(128, 3, (2045,), 0), (128, 3, (2046,), 0), (128, 3, (5000,), 16), (128, 3, (9000,), 0), (128, 3, (9300,), 16),
                                          (128, 9, (0, 2000, 63, 64), 16), (128, 9, (1, 9000, 700), 0), (64, 3, (2046,), 32), (64, 3, (11000,), 0),
                                          (64, 9, (0, 9000, 700), 16), (128, 1, (40,) * 70 + (6000,), 16), (128, 4, (3000,) * 6, 16), (128, 2, (9650, 9400), 16), (128, 2, (9650, 9500), 0),
                                          (128, 20, (8100, 7700), 0), (128, 20, (8100, 7800), 16)])
def test_shares_at_the_edges_of_the_work_split(d, n_q, L, page):
    # 8 KV heads: 256 granules of 64 keys and just above (a workgroup per granule; one per compute unit, units padded), just below and
    # above the point from which more workgroups than compute units take part (one per compute unit up to 16 rows: all of them), units
    # shorter than the padding beside long ones, and more sequences than a wave has lanes.  q.k is scaled up so that single keys decide and a lost or doubled tile shows.
    shape = gen.scaled(gen.config(1), B=len(L), Hq=8, Hkv=8, d=d, n_q=n_q, k=max(n_q - 1, 1), ctx=(0, 1), page_size=page or 16)
    L = np.array(L, np.int32)
    kv = gen.kv_cache(shape, L, n_q, 13, paged=page > 0)
    check(shape, L, kv, 4 * gen.queries(shape, 13), None, label="split edges")


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("d,n_q", [(128, 25), (128, 57), (64, 17), (64, 33)])
@pytest.mark.parametrize("L", [(5000, 4973, 5041), (2600, 2631, 2664, 2697, 3000), (700, 3001, 1234, 4100)])
def test_segments_around_the_depth_of_the_rings(d, n_q, page, L):
    # rings of four and eight slots, eight KV heads: segments of 4 to 11 granules with shorter ones at the units' ends, whose last tile
    # step has a tile for one ring or both, whole or not.  q.k is scaled up so that a lost or doubled tile shows.
    shape = gen.scaled(gen.config(1), B=len(L), Hq=16, Hkv=8, d=d, n_q=n_q, k=n_q - 1, ctx=(0, 1), page_size=page or 16)
    L = np.array(L, np.int32)
    kv = gen.kv_cache(shape, L, n_q, 17, paged=page > 0)
    rng = np.random.default_rng(n_q)
    only = [(b, int(i), int(rng.integers(16))) for b in range(len(L)) for i in (0, n_q // 2, n_q - 1) for _ in range(8)]
    check(shape, L, kv, 4 * gen.queries(shape, 17), None, only=only, label="ring depth")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,lengths,longest", [(1, (4090,), 4096), (1, (4111,), 4111), (1, (5610,), 5610), (1, (3900,), 5610), (1, (8150,), 8150), (2, (4000, 200), 4000),
                                               (3, (1500, 1600, 0), 1600), (5, (1000,) * 5, 1000), (8, (700,) * 8, 700)])
def test_shares_of_the_middle_range(dtype, B, lengths, longest):
    # four KV heads: up to 256 granules a workgroup each, from 257 on equal shares of two, of three; a cache that could hold more granules
    # than there are (the launch is sized for the cache), shares that are not all equal; five and eight sequences of one length, a whole
    # number of shares per unit
    shape = gen.scaled(gen.config(1), dtype=dtype, B=B, Hq=8, Hkv=4, d=64, n_q=3, ctx=(longest, longest))
    L, kv, q, mask = case(shape, 4)
    L[:] = lengths
    check(shape, L, kv, q, mask, label="middle range")


@pytest.mark.parametrize("dtype,n_q,page", [("f32", 8, 0), ("f32", 9, 0), ("f32", 17, 48), ("f32", 32, 0), ("bf16", 8, 48), ("bf16", 9, 48), ("f32", 1, 48), ("f32", 2, 0),
                                             ("f32", 16, 0), ("bf16", 16, 48), ("bf16", 17, 48)])
def test_alu_kernels_of_wide_heads(dtype, n_q, page):
    # four rows a query: 32 and 36 rows per KV head with accumulators for 32 and for 64, 64 and 68 in tiles of 64 and of 32 keys, the most
    # rows, and few whose keys the threads share
    shape = gen.scaled(gen.config(1), dtype=dtype, B=3, Hq=8, Hkv=2, d=128, n_q=n_q, k=max(n_q - 1, 1), ctx=(0, 400), page_size=page or 16)
    L, kv, q, mask = case(shape, 6, paged=page > 0)
    L[0] = 0
    check(shape, L, kv, q, mask, label="wide heads on the ALUs")


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("B,n_q", [(2, 3), (40, 7)])
def test_outputs_begin_at_any_element(dtype, d, B, n_q):
    # merged by a workgroup per row and by a wave per row: the output buffer asks for no alignment beyond its elements'
    shape = gen.scaled(gen.config(1), dtype=dtype, B=B, Hq=8, Hkv=2, d=d, n_q=n_q, ctx=(20, 400))
    L, kv, q, _ = case(shape, 9)
    lib = H.sx()
    view, keep = H.kv_view_of(shape, kv)
    qd, ctx = H.dev(q, shape), H.dev(L.astype(np.int32))
    ws = H.workspace(lib.specexit_verify_attn_workspace_bytes(view, B, n_q, shape.Hq))
    got = []
    for first in (0, 1, 2, 3):
        buf = torch.full((qd.numel() + 8,), 7.0, dtype=qd.dtype, device="cuda")
        out = buf[first:first + qd.numel()].view(qd.shape)
        lib.specexit_verify_attn(view, B, n_q, shape.Hq, qd, ctx, None, d ** -0.5, out, ws)
        torch.cuda.synchronize()
        assert bool((buf[:first] == 7.0).all()) and bool((buf[first + qd.numel():] == 7.0).all())
        got.append(H.host(out))
    for g in got[1:]:
        np.testing.assert_array_equal(g, got[0])


def test_paged_equals_contiguous_on_gpu():
    shape = gen.scaled(gen.config(2), B=4, Hq=8, Hkv=2, ctx=(30, 1200))
    L, kv, q, mask = case(shape, 3, paged=False)
    paged = gen.to_paged(shape, kv, shape.n_q, seed=1)
    a = gpu_verify_attn(shape, kv, q, L, mask)
    b = gpu_verify_attn(shape, paged, q, L, mask)
    np.testing.assert_array_equal(a, b)
    check(shape, L, paged, q, mask, label="paged")


@pytest.mark.parametrize("n_q,Hq,Hkv", [(1, 8, 2), (64, 4, 2), (16, 16, 2), (9, 8, 1)])
def test_block_size_extremes(n_q, Hq, Hkv):
    shape = gen.scaled(gen.config(1), B=2, Hq=Hq, Hkv=Hkv, n_q=n_q, k=min(5, max(n_q - 1, 1)), ctx=(50, 400))
    L, kv, q, mask = case(shape, 4, tree=n_q > 1)
    check(shape, L, kv, q, mask, label="extremes")


@pytest.mark.parametrize("n_q,Hq,Hkv", [(24, 8, 2), (25, 8, 2), (14, 16, 2), (29, 4, 1), (8, 16, 1)])
@pytest.mark.parametrize("page", [0, 16, 64])
def test_many_query_rows(n_q, Hq, Hkv, page):
    # 96 to 128 rows per KV head: from 97 on a wave takes two row tiles, the last of them ragged or empty
    shape = gen.scaled(gen.config(1), B=9, Hq=Hq, Hkv=Hkv, n_q=n_q, k=5, ctx=(0, 1500), page_size=page or 16)
    L, kv, q, mask = case(shape, 6, tree=page != 16, paged=page > 0)
    L[0], L[1] = 0, 1
    check(shape, L, kv, q, mask, label="many rows")


def test_self_only_mask_with_empty_context_returns_own_value():
    shape = gen.scaled(gen.config(1), B=2, Hq=4, Hkv=2, n_q=5, ctx=(0, 0))
    L, kv, q, _ = case(shape, 5)
    mask = np.array([[1 << i for i in range(5)]] * 2, dtype=np.uint64)
    got = gpu_verify_attn(shape, kv, q, L, mask)
    for i in range(5):
        for h in range(4):
            np.testing.assert_allclose(got[:, i, h], kv.v[:, h // 2, i], atol=1e-2)


def sample_triples(shape, n, seed):
    r = np.random.default_rng(seed)
    return [(int(r.integers(shape.B)), int(r.integers(shape.n_q)), int(r.integers(shape.Hq))) for _ in range(n)]


def test_full_size_config_1():
    shape = gen.config(1)
    L, kv, q, mask = case(shape, 0)
    check(shape, L, kv, q, mask, label="config 1 full")


@pytest.mark.parametrize("index", [2, 3, 4])
def test_full_size_sampled(index):
    """Full shapes; a sample of (sequence, query, head) outputs against the oracle."""
    shape = gen.config(index)
    L, kv, q, mask = case(shape, 0, tree=shape.tree)
    only = sample_triples(shape, 48, index)
    only += [(int(np.argmax(L)), shape.n_q - 1, 0), (int(np.argmin(L)), 0, shape.Hq - 1)]
    check(shape, L, kv, q, mask, only=only, label=f"config {index} sampled")


@pytest.mark.parametrize("n_q,Hq,d,page", [(1, 2, 128, 0), (1, 8, 128, 16), (4, 8, 128, 0), (4, 8, 64, 64), (2, 16, 64, 0), (5, 6, 128, 32)])
@pytest.mark.parametrize("B", [9, 64, 65])
def test_few_rows_at_ring_and_share_edges(B, n_q, Hq, d, page):
    # up to 16 rows per KV head: four rings of one wave, of which some have no tile, one or several, in segments that end inside a
    # unit or go on with the next.  64 sequences are the most whose lengths a workgroup's first segment takes from its lanes; the other
    # segments, and more sequences, take them from the table.
    shape = gen.scaled(gen.config(1), B=B, Hq=Hq, Hkv=2, d=d, n_q=n_q, k=max(n_q - 1, 1), ctx=(0, 700), page_size=page or 16)
    L, kv, q, mask = case(shape, 17, tree=n_q == 4, paged=page > 0)
    for b, n in enumerate((0, 31, 32, 33, 96, 97, 128, 129, 256)):
        L[b] = n
    err = check(shape, L, kv, q, mask, label=f"few rows, d {d} page {page}")
    assert err < 2.0 ** -8          # two-part probabilities: the bf16 rounding of the output, at most 2^-9 of the largest value
