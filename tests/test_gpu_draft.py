"""GPU parity: specexit_draft_step against the oracle."""
import numpy as np
import pytest

from oracle import specexit_oracle as O
from workloads import gen

from harness import TOL, GpuDraft, force_draft_gap, oracle_dims, oracle_draft_rows, rel_err

pytestmark = pytest.mark.gpu


def setup(shape, seed, paged=False, norms=True, std=0.02):
    w = gen.draft_weights(shape, seed, std=std)
    if norms:
        w.update(gen.perturbed_norm_vectors(shape, seed))
    pos = gen.context_lengths(shape, seed)
    kv = gen.kv_cache(shape, pos, shape.k + 1, seed, paged=paged)
    tok = gen.token_ids(shape, shape.B, seed)
    g = gen.hidden_rows(shape, shape.B, seed)
    return w, kv, tok, g, pos


def one_step(shape, w, kv, tok, g, pos, gd=None, label=""):
    print(f"draft_step {label}: dtype={shape.dtype} B={shape.B} D={shape.D} I={shape.I} V={shape.V} "
          f"pos={pos.tolist()[:8]} paged={kv.paged}", flush=True)
    kc, vc = kv.k.astype(np.float64), kv.v.astype(np.float64)
    ref = O.draft_step(oracle_dims(shape), w, kc, vc, tok, g, pos, kv.page_table if kv.paged else None,
                       kv.page_size, store=lambda a: gen.store(shape, a.astype(np.float32)))
    assert O.top2_gap(ref["logits"]).min() > 0.05
    gd = gd or GpuDraft(shape, w, kv)
    got = gd.step(tok, g, pos)
    tol = TOL[shape.dtype]
    np.testing.assert_array_equal(got["next_tok"], ref["next_tok"])
    assert rel_err(got["hidden_out"], ref["hidden_out"]) < tol
    assert rel_err(got["sig_raw"], ref["sig_raw"]) < tol
    assert rel_err(got["sig"][:, :2], ref["sig"][:, :2]) < tol
    assert rel_err(got["sig"][:, 2], ref["sig"][:, 2]) < tol
    # the cache entry written at pos
    gk, gv = gd.cache()
    for b in range(shape.B):
        p = int(pos[b])
        if kv.paged:
            pg, sl = kv.page_table[b, p // kv.page_size], p % kv.page_size
            assert rel_err(gk[pg, :, sl], kc[pg, :, sl]) < tol and rel_err(gv[pg, :, sl], vc[pg, :, sl]) < tol
        else:
            assert rel_err(gk[b, :, p], kc[b, :, p]) < tol and rel_err(gv[b, :, p], vc[b, :, p]) < tol
    return ref, got, gd, (kc, vc)


def test_tiny_fp32_config_chain_of_steps():
    shape = gen.config(0)
    w, kv, tok, g, pos = setup(shape, 0)
    gd = None
    for step in range(shape.k):
        w2 = force_draft_gap(shape, w, kv, tok, g, pos)
        if gd is None or not np.array_equal(w2["w_head"], w["w_head"]):
            gd = None                      # weights changed: rebuild the device copy (cache contents carry over)
        w = w2
        ref, got, gd, (kc, vc) = one_step(shape, w, kv, tok, g, pos, gd, label=f"config 0 step {step}")
        kv.k[:], kv.v[:] = kc, vc           # oracle's cache after the step feeds the next one
        tok = ref["next_tok"].astype(np.int32)
        g = ref["hidden_out"].astype(np.float32)
        pos = pos + 1
        gd = None


@pytest.mark.parametrize("B,D,I,V,paged", [(1, 256, 256, 257, True), (2, 512, 1280, 1000, False), (3, 256, 768, 3001, False), (4, 512, 256, 64, True),
                                           (5, 256, 512, 100, False), (8, 768, 2816, 5001, True), (9, 256, 5120, 2000, False), (17, 512, 512, 301, False), (26, 256, 3328, 500, False), (26, 256, 3072, 500, True),
                                           (2, 320, 512, 1000, False)])
def test_fp32_rows(B, D, I, V, paged):
    # one, two, four and eight rows per workgroup and their remainders; one to many steps of 256 weights; odd and even numbers of head
    # rows; the last one has no multiple of 256 and takes the plain kernels, as does one of many rows and a long K.  Tolerance: 32-bit sums (rel_err's limit of fp32 storage)
    shape = gen.scaled(gen.config(0), D=D, Hq=4, Hkv=2, d=64 if B % 2 else 128, I=I, V=V, B=B, ctx=(0, 200), k=2)
    w, kv, tok, g, pos = setup(shape, B, paged=paged, std=0.05)
    pos[0] = 0
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    one_step(shape, w, kv, tok, g, pos, label="fp32 rows")


@pytest.mark.parametrize("dtype,B,D", [("bf16", 1, 5120), ("bf16", 2, 5120), ("f32", 1, 4352), ("f32", 3, 4608)])
def test_sums_of_squares_in_more_pieces_than_256(dtype, B, D):
    # the row stream adds a piece per workgroup of the projection in front: 288 to 512 here, of bf16 models all requested together, of fp32
    # ones those beyond 256 by a loop.  With w_o = 0 no 16-bit value stands between the inputs and the signals, so they are 32-bit sums for
    # bf16 models too: one piece of 512 left out or taken twice is 1e-3 of 1 / rms.
    shape = gen.scaled(gen.config(4 if dtype == "bf16" else 0), D=D, Hq=4, Hkv=2, d=128, I=512, V=500, B=B, ctx=(0, 60), k=2)
    w, kv, tok, g, pos = setup(shape, B, std=0.05)
    w["w_o"] = np.zeros_like(w["w_o"])
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    ref, got, _, _ = one_step(shape, w, kv, tok, g, pos, label="pieces")
    assert rel_err(got["sig_raw"], ref["sig_raw"]) < TOL["f32"]


@pytest.mark.parametrize("B,paged", [(1, False), (2, True), (3, True), (9, False), (16, True)])
def test_small_bf16_mfma(B, paged):
    shape = gen.scaled(gen.config(2), D=256, Hq=4, Hkv=2, d=64, I=512, V=3000, B=B, ctx=(0, 300), k=2)
    w, kv, tok, g, pos = setup(shape, B, paged=paged, std=0.05)
    pos[0] = 0
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    one_step(shape, w, kv, tok, g, pos, label="small mfma")


@pytest.mark.parametrize("B,D", [(17, 512), (32, 512), (33, 512), (49, 512), (64, 512), (20, 2048), (40, 2048)])
def test_row_tile_edges(B, D):
    # (weight rows 4 KB apart, D = 2048: the head sums K in two chunks)
    shape = gen.scaled(gen.config(2), D=D, Hq=4, Hkv=2, d=128, I=768, V=3001, B=B, ctx=(0, 60), k=2)
    w, kv, tok, g, pos = setup(shape, B, std=0.05)
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    one_step(shape, w, kv, tok, g, pos, label="row tile edges")


@pytest.mark.parametrize("Hq,d,page", [(2, 128, 0), (8, 128, 16), (32, 128, 32), (8, 64, 64), (32, 64, 0)])
@pytest.mark.parametrize("B,L", [(9, (0, 31, 32, 33, 96, 97, 128, 129, 256)), (40, (64, 1, 700, 127)), (3, (9000, 1, 2047))])
def test_attention_of_few_rows_at_ring_and_share_edges(B, L, Hq, d, page):
    # draft steps have two rings, of one wave up to 16 rows per KV head: rings without a tile, with one or several, segments that end inside
    # a unit or go on with the next, shares of one granule and of many
    shape = gen.scaled(gen.config(2), D=256, Hq=Hq, Hkv=2, d=d, I=512, V=1000, B=B, ctx=(0, 500), k=2, page_size=page or 16)
    w, kv, tok, g, pos = setup(shape, 19, std=0.05)
    pos[:len(L)] = L
    kv = gen.kv_cache(shape, pos, shape.k + 1, 19, paged=page > 0)
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    one_step(shape, w, kv, tok, g, pos, label=f"few rows, d {d} page {page}")


@pytest.mark.parametrize("B", [5, 20])
@pytest.mark.parametrize("D,I", [(256, 8192), (1024, 1024), (128, 16384)])
def test_sums_over_few_and_many_slots(B, D, I):
    # partial sums of a projection in two to more than eight places: many groups of few k blocks (gate and up), few groups of many (down),
    # rows of more than one float4 per thread excepted, which the full-size cases have
    shape = gen.scaled(gen.config(2), D=D, Hq=2, Hkv=1, d=128, I=I, V=500, B=B, ctx=(0, 60), k=2)
    w, kv, tok, g, pos = setup(shape, B, std=0.05)
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    one_step(shape, w, kv, tok, g, pos, label="slots")


@pytest.mark.parametrize("B,V", [(20, 98400), (33, 151936), (20, 165001), (64, 82000), (64, 151936)])
def test_head_passes_of_several_halves(B, V):
    # the widened head over two planes: four and five halves in a pass, twice three; three, three and two of four row tiles
    shape = gen.scaled(gen.config(2), D=256, Hq=4, Hkv=2, d=64, I=256, V=V, B=B, ctx=(0, 60), k=2)
    w, kv, tok, g, pos = setup(shape, B, std=0.05)
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    one_step(shape, w, kv, tok, g, pos, label="head passes")


@pytest.mark.parametrize("B", [5, 9, 40])
def test_odd_number_of_narrow_kv_heads(B):
    # the k block and the v block of the q|k|v projection then begin inside a group of 128 rows
    shape = gen.scaled(gen.config(2), D=256, Hq=6, Hkv=3, d=64, I=384, V=1000, B=B, ctx=(0, 60), k=2)
    w, kv, tok, g, pos = setup(shape, B, std=0.05)
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    one_step(shape, w, kv, tok, g, pos, label="odd kv heads")


def known_rows(D, B, seed):
    """A step whose normed rows are known to the last bit: the layer passes the integers of hidden_in through (W_fc = [0 | 1], no
    attention, no MLP), and their squares add up exactly in any order.  Returns the step's inputs, the normed rows in
    32 bits and in 64, and the head's rows."""
    shape = gen.scaled(gen.config(2), D=D, Hq=4, Hkv=2, d=128, I=512, V=500, B=B, ctx=(5, 20), k=2)
    rng = np.random.default_rng(1000 * seed + B)
    w = gen.draft_weights(shape, seed)
    w["w_fc"] = np.concatenate([np.zeros((D, D), np.float32), np.eye(D, dtype=np.float32)], 1)
    w["w_o"], w["w_down"] = np.zeros_like(w["w_o"]), np.zeros_like(w["w_down"])
    gain = w["ln_final"] = gen.store(shape, rng.uniform(0.5, 1.5, D).astype(np.float32))
    g = (rng.integers(1, 16, (B, D)) * rng.choice([-1, 1], (B, D))).astype(np.float32)
    pos = gen.context_lengths(shape, seed)
    gd = GpuDraft(shape, w, gen.kv_cache(shape, pos, shape.n_q, seed))
    mean = (g.astype(np.float64) ** 2).mean(1, keepdims=True)
    assert D & (D - 1) == 0 and mean.max() * D < 2 ** 24
    n32 = g * (np.float32(1) / np.sqrt(mean.astype(np.float32) + np.float32(shape.rms_eps))) * gain
    n64 = g * gain.astype(np.float64) / np.sqrt(mean + np.float64(np.float32(shape.rms_eps)))
    return gd, (gen.token_ids(shape, B, seed), g, pos), n32, n64, w["w_head"].astype(np.float64)


@pytest.mark.parametrize("B", [5, 16, 17, 40, 64])
def test_sums_of_two_part_rows(B):
    # The head's sums over K = 4096, given the two bf16 parts of the rows.  n roundings at the size of the sum so far, whose square grows
    # evenly, add up to 2^-24 sqrt(n / 2) of the result.  Up to 16 rows: four chunks of half the size, 32 products of the
    # values each, 4 (1/2)^2 32 / 2 = 16; the rest adds up by itself.  More rows: 32 blocks are added, 32 / 2 = 16, and in
    # each 8 products of either part at 32^-1/2 of the size, 8 / 2 = 4 together.  (Both parts in one sum over all of K: 128.)
    bound = 2.0 ** -24 * (16 if B <= 16 else 20) ** 0.5
    err = []
    for seed in range(4):
        gd, (tok, g, pos), n32, _, head = known_rows(4096, B, seed)
        hi = gen.round_to_bf16(n32)
        parts = hi.astype(np.float64) + gen.round_to_bf16(n32 - hi)
        got = gd.tree(tok, g, pos, np.array([-1, 0], np.int32), np.zeros(2, np.int32), 4)
        ref = np.einsum("bd,bvd->bv", parts, head[got["cand_tok"][0]])
        err.append((got["cand_logit"][0] - ref) / ref)
    err = np.sqrt((np.concatenate(err) ** 2).mean())
    print(f"  {B} rows: {err:.2e} of {bound:.2e}", flush=True)
    assert err < bound


@pytest.mark.parametrize("B", [1, 2, 3, 4])
def test_steps_of_few_rows_keep_32_bits(B):
    # Steps of up to four rows multiply 32-bit values.  Sums of 2048 products in 32 bits, 32 of them in a row in each of 64 lanes, are
    # off by 2^-24 sqrt(32 / 2) 0.4 = 1e-7 of their size, the rows' factor by 2^-24 at most; taken as two bf16 parts, the operands
    # themselves would be off by some 2^-9 of 2^-9, 1.2e-6.
    err = []
    for seed in range(8):
        gd, inputs, _, n64, head = known_rows(2048, B, seed)
        ref = n64 @ head[gd.shape.V:].T
        err.append((gd.step(*inputs)["sig_raw"] - ref) / (np.linalg.norm(n64, axis=1, keepdims=True) * head.std()))
    err = np.sqrt((np.concatenate(err) ** 2).mean())
    print(f"  {B} rows: {err:.2e}", flush=True)
    assert err < 4e-7


def test_small_bf16_alu_fallback():
    shape = gen.scaled(gen.config(1), D=192, Hq=4, Hkv=2, d=64, I=320, V=1000, B=2, ctx=(5, 90), k=2)
    w, kv, tok, g, pos = setup(shape, 1, std=0.05)
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    one_step(shape, w, kv, tok, g, pos, label="small alu bf16")


def test_rem_activation_variants():
    shape = gen.scaled(gen.config(0), V=512)
    w, kv, tok, g, pos = setup(shape, 2)
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    raw = GpuDraft(shape, w, kv, rem_activation=2).step(tok, g, pos)
    sg = GpuDraft(shape, w, kv, rem_activation=1).step(tok, g, pos)
    np.testing.assert_allclose(raw["sig"][:, 2], raw["sig_raw"][:, 2], rtol=1e-6)
    np.testing.assert_allclose(sg["sig"][:, 2], 1 / (1 + np.exp(-sg["sig_raw"][:, 2].astype(np.float64))), rtol=1e-5)


def test_full_size_config_1():
    shape = gen.config(1)
    w, kv, tok, g, pos = setup(shape, 0, norms=False)
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    ref, got, gd, _ = one_step(shape, w, kv, tok, g, pos, label="config 1 full size")
    # the launch configuration bench.py times: workspace zero-filled once, flag set; same bits,
    # call after call
    prep = GpuDraft(shape, w, kv)
    prep.lib.specexit_workspace_prepare(prep.ws)
    for it in range(6):
        out = prep.step(tok, g, pos, flags=prep.lib.FLAG_WORKSPACE_PREPARED)
        for k in out:
            np.testing.assert_array_equal(out[k], got[k], err_msg=f"prepared call {it}: {k}")


def sampled_rows_step(shape, w, kv, tok, g, pos, rows, label):
    """The step runs over all B rows on the GPU; the oracle computes the sampled rows (rows of a step are
    independent of one another) and those are compared: token bit-exact, floats within tolerance."""
    print(f"draft_step {label}: dtype={shape.dtype} B={shape.B} D={shape.D} I={shape.I} V={shape.V} "
          f"pos={pos.tolist()} paged={kv.paged} oracle rows={rows}", flush=True)
    gd = GpuDraft(shape, w, kv)                       # device copies are taken before the oracle writes its entries
    got = gd.step(tok, g, pos)
    gk, gv = gd.cache()
    ref = oracle_draft_rows(shape, w, kv, tok, g, pos, rows, progress=label)
    tol = TOL[shape.dtype]
    for b in rows:
        r = ref[b]
        assert O.top2_gap(r["logits"][None, :])[0] > 0.05
        assert got["next_tok"][b] == O.argmax_lowest(r["logits"]), f"row {b}"
        assert rel_err(got["hidden_out"][b], r["hidden_out"]) < tol, f"row {b}"
        assert rel_err(got["sig_raw"][b], r["sig_raw"]) < tol, f"row {b}"
        assert rel_err(got["sig"][b], O.signal_activations(r["sig_raw"][None, :])[0]) < tol, f"row {b}"
        p = int(pos[b])
        if kv.paged:
            pg, sl = kv.page_table[b, p // kv.page_size], p % kv.page_size
            assert rel_err(gk[pg, :, sl], kv.k[pg, :, sl]) < tol and rel_err(gv[pg, :, sl], kv.v[pg, :, sl]) < tol
        else:
            assert rel_err(gk[b, :, p], kv.k[b, :, p]) < tol and rel_err(gv[b, :, p], kv.v[b, :, p]) < tol
    assert np.isfinite(got["hidden_out"]).all() and (got["next_tok"] >= 0).all() and (got["next_tok"] < shape.V).all()


@pytest.mark.timeout(1500)
def test_full_size_config_2_all_eight_rows():
    """Qwen3-8B-like sizes, B = 8, paged cache: the split-K matrix-core projections with their reducing
    epilogues at full width (steps of few rows take the row-streaming path); every row compared."""
    shape = gen.config(2)
    w, kv, tok, g, pos = setup(shape, 0, paged=True, norms=False)
    rows = list(range(shape.B))
    w = force_draft_gap(shape, w, kv, tok, g, pos, rows=rows)
    sampled_rows_step(shape, w, kv, tok, g, pos, rows, "config 2 full size")


@pytest.mark.timeout(1500)
def test_full_size_config_4_sixteen_rows():
    """32B-like sizes (D = 5120, I = 25600, 64 query heads, paged caches of 8k-32k entries), B = 16 rows in
    the launch shapes bench.py times; the oracle checks the longest and the shortest sequence's rows and one more."""
    shape = gen.config(4)
    w, kv, tok, g, pos = setup(shape, 0, paged=True, norms=False)
    rows = sorted({int(np.argmax(pos)), int(np.argmin(pos)), 7})
    w = force_draft_gap(shape, w, kv, tok, g, pos, rows=rows)
    sampled_rows_step(shape, w, kv, tok, g, pos, rows, "config 4 full size")


def test_prepared_workspace_flag_gives_the_same_results_call_after_call():
    """The flag promises a workspace that was zero-filled once and then kept to this call.  No kernel needs that
    today: with and without it, call after call, the results are the same."""
    shape = gen.scaled(gen.config(2), D=512, Hq=8, Hkv=2, d=128, I=1024, V=5000, B=3, ctx=(10, 400), k=2)
    w, kv, tok, g, pos = setup(shape, 7, std=0.05)
    w = force_draft_gap(shape, w, kv, tok, g, pos)
    plain = GpuDraft(shape, w, kv)
    prep = GpuDraft(shape, w, kv)
    prep.ws.fill_(0x5A)                                   # garbage first: prepare must clear it
    prep.lib.specexit_workspace_prepare(prep.ws)
    for it in range(12):
        a = plain.step(tok, g, pos + it % 3)
        b = prep.step(tok, g, pos + it % 3, flags=prep.lib.FLAG_WORKSPACE_PREPARED)
        for k in a:
            np.testing.assert_array_equal(a[k], b[k], err_msg=f"call {it} {k}")


def test_reducing_epilogues_give_identical_bits_every_time():
    """Partial sums over K ranges are added in their order, whichever workgroup finished first:
    forty repetitions of one step (six rows: the matrix-core path) must agree bit for bit,
    outputs and cache entry alike."""
    shape = gen.scaled(gen.config(2), D=1024, Hq=8, Hkv=2, d=128, I=2560, V=9000, B=6, ctx=(100, 900), k=2)
    w, kv, tok, g, pos = setup(shape, 11, paged=True, std=0.05)
    gd = GpuDraft(shape, w, kv)
    first, cache0 = None, None
    for it in range(40):
        out = gd.step(tok, g, pos)
        gk, gv = gd.cache()
        if first is None:
            first, cache0 = out, (gk, gv)
            continue
        for k in out:
            np.testing.assert_array_equal(out[k], first[k], err_msg=f"repetition {it}: {k}")
        np.testing.assert_array_equal(gk, cache0[0])
        np.testing.assert_array_equal(gv, cache0[1])
