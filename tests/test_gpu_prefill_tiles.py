"""The ring kernel of the prompt GEMMs: every tile shape and K split against the chunked prompt pass (the decode kernels).

pf_ring=V names a shape by number: in bf16 2 is the largest (16 weight tiles or 8 pairs x 16 chunks), 0 and 1 are 16 x 8 and 12 x 8 tiles (8 and 12 pairs x 8), 3 the
smallest of QKV and the raw sums (4 x 2; gate/up 4 pairs x 5), 4 to 15 lie between; in fp32 3 is the largest and 4 the smallest (3 x 2).

The first two shapes have output widths that no tile divides (feature blocks with a partly filled last tile, and fewer blocks than
XCDs), and K ranges shorter than the ring; their workspace holds 512 rows.  The other two have a vocabulary large enough for the
staging region to hold blocks of 1024 and 2048 rows.  The prompts end inside a 16-row chunk, inside a workgroup's 8 (16) chunks,
and inside the first, second and third block.  Both paths hold activations as two bf16 planes and sum in fp32; they differ in the order of the sums, and K / V values next to a bf16
rounding boundary then differ by one unit: TOL of the parity tests."""
import numpy as np
import pytest

import asd_inputs as si
import paper_2410_01028_amd as asd
from test_gpu_parity import COS_TOL, TOL, rel_err

pytestmark = pytest.mark.gpu

# 24 QKV tiles, 14 residual tiles, 21 gate/up pairs; k-blocks 7 (odd), 6, 11 (odd, the last half padding)
RAGGED = si.Shape("ragged", 2, 224, 6, 3, 32, 336, 320, si.DT_BF16, 8, 8, 2)
EVEN = si.Shape("even", 2, 320, 4, 2, 64, 512, 320, si.DT_BF16, 8, 8, 2)
LONG_1K = si.Shape("long-1k", 2, 256, 4, 2, 64, 256, 6016, si.DT_BF16, 8, 8, 2)
LONG_2K = si.Shape("long-2k", 2, 256, 12, 4, 32, 256, 18944, si.DT_BF16, 8, 8, 2)       # from 1921 rows: the long-block attention
LEAST = si.Shape("least", 1, 16, 1, 1, 32, 16, 16, si.DT_BF16, 8, 8, 2)      # one tile, one k-block, half of it padding
LONGEST = {"least": 512, "ragged": 512, "even": 512, "long-1k": 1024, "long-2k": 2048}
CASES = [(RAGGED, "pf_ring=0", 81), (RAGGED, "pf_ring=1", 130), (RAGGED, "pf_ring=2,2", 97), (RAGGED, "pf_ring=3", 300), (RAGGED, "pf_ring=0,6", 200),
         (RAGGED, "pf_ring=4", 17), (RAGGED, "pf_ring=5", 45), (RAGGED, "pf_ring=6", 63), (RAGGED, "pf_ring=7,1", 100), (RAGGED, "pf_ring=8", 33),
         (RAGGED, "pf_ring=9,3", 49), (RAGGED, "pf_ring=10", 81), (RAGGED, "pf_ring=11", 128), (RAGGED, "pf_ring=12", 32), (RAGGED, "pf_ring=13", 40),
         (RAGGED, "pf_ring=14", 64), (RAGGED, "pf_ring=15,5", 144), (RAGGED, "pf_ring=2", 300), (EVEN, None, 18), (EVEN, None, 300), (EVEN, "pf_ring=1,8", 500),
         (EVEN, "pf_ring=2,1", 144), (EVEN, "pf_ring=3,2", 1000), (EVEN, None, 2049), (EVEN, "pf_ring=3,1", 2300), (EVEN, "pf_ring=2,2", 1000), (EVEN, "pf_ring=2,1", 2300), (EVEN, "pf_o=4,4,2", 1500),
         (LEAST, None, 17), (LEAST, None, 600), (LEAST.with_(dtype=si.DT_F32), None, 45), (LONG_1K, None, 641), (LONG_1K, None, 1003), (LONG_1K, None, 1025), (LONG_1K, None, 2300), (LONG_1K, "pf_ring=1,4", 1009),
         (LONG_1K, "pf_o=4,4,2;pf_down=8,3,2;pf_qkv=4,1,2;pf_gu=4,1,2", 1700), (LONG_2K, None, 641), (LONG_2K, None, 1003), (LONG_2K, None, 2041),
         (LONG_2K, None, 2049), (LONG_2K, None, 4001), (LONG_2K, None, 4200), (LONG_2K, "pf_ring=3,2", 2035), (LONG_2K, "pf_ring=2,2", 2035), (LONG_2K, "pf_ring=2,1", 2300), (LONG_2K, "pf_ring=15,3", 1345),
         (LONG_2K, "pf_ring=13", 700), (LONG_2K, "pf_o=4,4,2;pf_down=4,4,2;pf_qkv=4,1,2;pf_gu=4,1,2", 1985)]


@pytest.mark.parametrize("shape,tune,n", CASES, ids=[f"{s.name}-{s.dtype}-{t}-{n}" for s, t, n in CASES])
def test_prompt_gemm_tiles_agree_with_the_chunked_pass(shape, tune, n):
    W = list(si.all_tensors(shape, 6, 0.1))
    cfg = asd.make_config(shape, n + 16, debug_tune=tune)
    plan = asd.plan_prompt(cfg, n)
    assert len(plan) == -(-n // LONGEST[shape.name])
    if tune and tune.startswith("pf_ring"):
        want = tune[len("pf_ring="):].split(",")
        assert all(set(b["tile"].values()) == {int(want[0])} for b in plan)
        assert len(want) == 1 or all(b["slices"][g] == int(want[1]) for b in plan for g in ("oproj", "down"))
    assert shape is not LONG_2K or [b["attn_rows"] for b in plan] == [128 if b["rows"] > 1920 else 16 for b in plan]
    eng = asd.Engine(cfg).load(W)
    ref = asd.Engine(asd.make_config(shape, n + 16)).load(W)
    toks = si.prompt(n, n + 3, shape.vocab)
    _, acs, lg = eng.prefill(toks[:n], want_logits=True)
    _, acs2, lg2 = ref.prefill(toks[:n], want_logits=True, chunked=True)
    assert eng.kv_len == n and np.abs(acs - acs2).max() < COS_TOL
    assert rel_err(lg, lg2) < TOL[shape.dtype]
    a = eng.forward(toks[n:n + 3], n)["logits"]
    b = ref.forward(toks[n:n + 3], n)["logits"]
    assert rel_err(a, b).max() < TOL[shape.dtype]
    for l in range(shape.n_layers):
        k, v = eng.get_kv(l, 0, n)
        k2, v2 = ref.get_kv(l, 0, n)
        for x, y in ((k, k2), (v, v2)):
            assert np.abs(x - y).max() <= 2 ** -7 * np.abs(y).max()          # one bf16 unit at the largest value
            assert np.linalg.norm(x - y) < 1e-3 * np.linalg.norm(y)
    eng.close(); ref.close()


@pytest.mark.parametrize("shape,n", [(RAGGED, 17), (RAGGED, 45), (RAGGED, 100), (RAGGED, 520), (RAGGED, 640), (LONG_2K, 517), (LONG_2K, 640)],
                         ids=lambda v: getattr(v, "name", str(v)))
def test_tile_shape_does_not_enter_the_bits(shape, n):
    """With equal K slices (blocks of up to 640 rows) a prompt's logits, cosines and cache are the same bits in every tile shape and in
    the four-wave kernel."""
    toks = si.prompt(n, n, shape.vocab)
    W = list(si.all_tensors(shape, 2, 0.1))
    got = []
    for tune in ("pf_qkv=4,1,2;pf_o=4,4,2;pf_gu=4,1,2;pf_down=4,4,2", None, "pf_ring=0,4", "pf_ring=2,4", "pf_ring=3,4", "pf_ring=5,4", "pf_ring=11,4"):
        cfg = asd.make_config(shape, n + 16, debug_tune=tune)
        assert all(b["slices"]["oproj"] == b["slices"]["down"] == 4 for b in asd.plan_prompt(cfg, n))
        eng = asd.Engine(cfg).load(W)
        got.append((*eng.prefill(toks, want_logits=True), *eng.get_kv(1, 0, n)))
        eng.close()
    for g in got[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(got[0], g))


# head_dim, heads, KV heads, prompt, query rows per attention workgroup in each (512-row) block: 128 from 192 such workgroups on.
# Every head dim with and without grouped queries, last blocks that end inside a 16-row chunk, a wave's 32 rows and a
# workgroup's 128, and blocks too short for the long-block kernel behind long ones
LONG = [(32, 48, 48, 902, [128, 128]), (32, 64, 8, 949, [128, 128]), (64, 48, 6, 900, [128, 128]), (64, 56, 56, 985, [128, 128]),
        (128, 48, 48, 911, [128, 128]), (128, 64, 8, 1001, [128, 128]), (128, 48, 8, 1412, [128, 128, 128]), (32, 64, 64, 513, [128, 16]),
        (128, 64, 8, 2177, [128] * 4 + [16]), (32, 32, 8, 1030, [16, 16, 16])]


@pytest.mark.parametrize("h,n_h,n_kv,n,attn_rows", LONG, ids=lambda v: str(v))
def test_long_block_attention_agrees_with_the_chunked_pass(h, n_h, n_kv, n, attn_rows):
    shape = si.Shape("wide", 2, 256, n_h, n_kv, h, 256, 256, si.DT_BF16, 8, 8, 2)
    assert [b["attn_rows"] for b in asd.plan_prompt(asd.make_config(shape, n + 16), n)] == attn_rows
    W = list(si.all_tensors(shape, 11, 0.1))
    # larger q and k weights: scores of several units, so that running maxima move and rows have few heavy keys
    W = [(t, l, si_scale(a, 3.0) if t in (si.T_WQ, si.T_WK) else a) for t, l, a in W]
    eng = asd.Engine(asd.make_config(shape, n + 16)).load(W)
    ref = asd.Engine(asd.make_config(shape, n + 16)).load(W)
    pages = -(-(n + 16) // 64)
    for e in (eng, ref):
        e.set_page_table(np.random.default_rng(n).permutation(pages))
    toks = si.prompt(n, n + 3, shape.vocab)
    _, acs, lg = eng.prefill(toks[:n], want_logits=True)
    _, acs2, lg2 = ref.prefill(toks[:n], want_logits=True, chunked=True)
    assert np.abs(acs - acs2).max() < COS_TOL
    assert rel_err(lg, lg2) < TOL[shape.dtype]
    k, v = eng.get_kv(1, 0, n)          # the second layer's cache carries every row's attention output of the first
    k2, v2 = ref.get_kv(1, 0, n)
    for x, y in ((k, k2), (v, v2)):
        assert np.linalg.norm(x - y) < 1e-3 * np.linalg.norm(y)
    eng.close(); ref.close()


def test_rows_whose_first_keys_all_score_minus_infinity():
    """Scores that overflow to -inf count for nothing, whichever attention kernel takes the row: 70 tokens A, then tokens B whose
    scores against every A are -inf and against every B zero, so that the first key chunk of every B row holds nothing.  192
    workgroups of 128 rows: the long-block kernel."""
    n, n_a = 450, 70
    shape = si.Shape("wide", 2, 256, 48, 48, 32, 256, 256, si.DT_BF16, 8, 8, 2)
    assert [b["attn_rows"] for b in asd.plan_prompt(asd.make_config(shape, n + 16), n)] == [128]
    W = {(t, l): a.copy() for t, l, a in si.all_tensors(shape, 5, 0.1)}
    bf16 = lambda x: np.uint16(np.float32(x).view(np.uint32) >> 16)
    emb = W[si.T_EMBED, 0]
    emb[:2] = 0
    emb[0, 0] = emb[1, 1] = bf16(1.0)                      # token 0 (A) is feature 0, token 1 (B) feature 1; 16 each behind the norm
    W[si.T_ATTN_NORM, 0][:] = 1.0
    for t, col, val in ((si.T_WQ, 1, -1e19), (si.T_WK, 0, 1e19)):
        w = W[t, 0]
        w[:, :2] = 0
        w[15::32, col] = bf16(val)                         # the slowest rotary pair: 0.08 radians over the prompt
    toks = np.where(np.arange(n + 3) < n_a, 0, 1).astype(np.int32)
    got = []
    for chunked in (False, True):
        eng = asd.Engine(asd.make_config(shape, n + 16)).load([(t, l, a) for (t, l), a in W.items()])
        _, acs, lg = eng.prefill(toks[:n], want_logits=True, chunked=chunked)
        got.append((acs, lg, *eng.get_kv(1, 0, n), eng.forward(toks[n:], n)["logits"]))
        eng.close()
    a, b = got
    assert all(np.isfinite(x).all() for x in a) and np.abs(a[0] - b[0]).max() < COS_TOL
    assert rel_err(a[1], b[1]) < TOL[shape.dtype] and rel_err(a[4], b[4]).max() < TOL[shape.dtype]
    for x, y in zip(a[2:4], b[2:4]):
        assert np.linalg.norm(x - y) < 1e-3 * np.linalg.norm(y)


def si_scale(a, f):
    """bf16 bit patterns times f, rounded to nearest even."""
    x = (si.bf16_to_f32(a) * np.float32(f)).view(np.uint32)
    return ((x + 0x7fff + ((x >> 16) & 1)) >> 16).astype(np.uint16)


@pytest.mark.parametrize("shape,n", [(LONG_1K, 1021), (LONG_1K, 1500), (LONG_2K, 2043), (LONG_2K, 2600)], ids=lambda v: getattr(v, "name", str(v)))
def test_weights_survive_prompt_blocks_laid_over_the_staging_region(shape, n):
    """Long blocks share memory with the region weight uploads go through: uploads and read-backs between prompt passes
    leave each other's results alone, and so does whatever the arena held before (rows past the prompt's end stay unread)."""
    W = list(si.all_tensors(shape, 3))
    cfg = asd.make_config(shape, n + 16)
    assert asd.plan_prompt(cfg, n)[0]["rows"] > 512
    eng = asd.Engine(cfg).load(W)
    toks = si.prompt(1, n, shape.vocab)
    run = lambda: (*eng.prefill(toks, want_logits=True), *eng.get_kv(1, 0, n))
    a = run()
    for t, l, arr in W:
        assert np.array_equal(eng.get_weight(t, l, arr.shape, arr.dtype), arr)
    b = run()
    eng.load(W)
    c = run()
    eng.close()
    eng = asd.Engine(cfg, arena_fill=0xFF).load(W)
    d = run()
    for x, *others in zip(a, b, c, d):
        assert all(np.array_equal(x, y) for y in others)
    eng.close()


F32_RAGGED = si.Shape("f32-ragged", 2, 176, 6, 3, 32, 272, 320, si.DT_F32, 8, 8, 2)


@pytest.mark.parametrize("n", [17, 33, 100, 300, 513])
def test_fp32_tile_shapes_give_the_same_bits(n):
    """The ring kernel on fp32 weights (k-blocks of 16, one plane): all tile shapes against the four-wave kernel bit for bit, and
    that against the chunked pass."""
    toks = si.prompt(n, n, F32_RAGGED.vocab)
    W = list(si.all_tensors(F32_RAGGED, 2, 0.1))
    got = []
    for tune in ("pf_qkv=4,1,2;pf_o=4,4,2;pf_gu=4,1,2;pf_down=4,4,2", None, "pf_ring=0,4", "pf_ring=1,4", "pf_ring=2,4", "pf_ring=3,4", "pf_ring=4,4",
                 "pf_ring=8,4", "pf_ring=11,4", "pf_ring=14,4"):
        eng = asd.Engine(asd.make_config(F32_RAGGED, n + 16, debug_tune=tune)).load(W)
        got.append((*eng.prefill(toks, want_logits=True), *eng.get_kv(1, 0, n)))
        if tune is None:
            ref = eng.prefill(toks, want_logits=True, chunked=True)
        eng.close()
    for g in got[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(got[0], g))
    assert np.abs(got[0][1] - ref[1]).max() < COS_TOL and rel_err(got[0][2], ref[2]) < TOL[si.DT_F32]


@pytest.mark.parametrize("d,ffn,n", [(16, 16, 17), (256, 688, 200), (272, 592, 45), (1024, 1040, 33)], ids=str)
def test_fp32_waves_on_their_own_give_the_same_bits(d, ffn, n):
    """pf_direct_kernel at one k-block, at a whole batch of requests, one past it and at four batches, with tiles that do not fill its workgroups, against the
    four-wave kernel; the estimate takes it where the slices are short and the launch has a compute unit per workgroup, and not beyond."""
    shape = si.Shape("direct", 2, d, 3, 3, 32, ffn, 320, si.DT_F32, 8, 8, 2)
    toks = si.prompt(n, n, shape.vocab)
    W = list(si.all_tensors(shape, 3, 0.1))
    got = []
    for tune in ("pf_qkv=4,1,2;pf_o=4,4,2;pf_gu=4,1,2;pf_down=4,4,2", None, "pf_ring=2"):
        cfg = asd.make_config(shape, n + 16, debug_tune=tune)
        tiles = asd.plan_prompt(cfg, n)[0]["tile"]
        if tune is None:
            assert tiles["qkv"] == 2 and (tiles["oproj"] == 2) == (n < 200)
        eng = asd.Engine(cfg).load(W)
        got.append((*eng.prefill(toks, want_logits=True), *eng.get_kv(1, 0, n)))
        eng.close()
    for g in got[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(got[0], g))
