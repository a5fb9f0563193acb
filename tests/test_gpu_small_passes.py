"""Decode passes of small fp32 models (one launch per sublayer) against the same passes as one launch per step (`small=0`): the
order of every sum is the same, so the bits are."""
import numpy as np
import pytest

import asd_inputs as si
import paper_2410_01028_amd as asd

pytestmark = pytest.mark.gpu

# edges of what the kernels take: features 64 .. 256 (odd numbers of tiles, a ragged last group of 64), 1 .. 8 heads of each size (16 and 32 dims per
# slice), hidden tiles that do not divide by the eight slices, a vocabulary whose last 64 and last 32 logits are not whole
SHAPES = [si.SHAPES["tiny"],
          si.Shape("one-head", 2, 64, 1, 1, 128, 128, 48, si.DT_F32, 8, 8, 2),
          si.Shape("two-heads", 2, 240, 2, 2, 128, 768, 336, si.DT_F32, 8, 8, 2),
          si.Shape("narrow", 3, 112, 4, 4, 32, 208, 400, si.DT_F32, 8, 8, 2),
          si.Shape("eight-heads", 2, 256, 8, 8, 32, 400, 1024, si.DT_F32, 8, 8, 2),
          si.Shape("two-small-heads", 1, 16, 2, 2, 64, 752, 16, si.DT_F32, 8, 8, 2)]


def engines(s, max_seq=1024):
    W = list(si.all_tensors(s, 5, gain_std=0.1))
    return [asd.Engine(asd.make_config(s, max_seq, page_tokens=64, debug_tune=t)).load(W) for t in (None, "small=0")]


def same(a, b, what):
    for k in a:
        assert np.array_equal(np.asarray(a[k]).view(np.int32), np.asarray(b[k]).view(np.int32)), (what, k)


@pytest.mark.parametrize("s", SHAPES, ids=lambda s: s.name)
def test_passes_have_the_bits_of_one_launch_per_step(s):
    """Every row count, over the edges of chunks, of the groups of 256 keys, and past the longest context of these kernels (768)."""
    new, old = engines(s)
    rng = np.random.default_rng(3)
    toks = rng.integers(0, s.vocab, 1024, dtype=np.int32)
    mask = np.zeros(2 * s.n_layers, np.uint8)
    for start, rows in ((0, (1, 2, 5, 9, 16, 3)), (57, (6, 7, 4, 1)), (250, (3, 8, 1)), (505, (13, 1, 4)), (751, (16, 1, 4, 1))):
        for e in (new, old):
            e.reset()
            for p in range(0, start, 16):
                e.forward(toks[p:min(start, p + 16)], p, want_logits=False)
        pos = start
        for n in rows:
            for skip in (None, mask):
                if skip is not None:
                    skip[:] = rng.integers(0, 2, skip.size)
                a, b = (e.forward(toks[pos:pos + n], pos, skip, commit=False) for e in (new, old))
                same(a, b, (start, pos, n, skip))
            a, b = (e.forward(toks[pos:pos + n], pos) for e in (new, old))
            same(a, b, (start, pos, n))
            pos += n
        for layer in range(s.n_layers):
            for x, y in zip(new.get_kv(layer, 0, pos), old.get_kv(layer, 0, pos)):
                assert np.array_equal(x.view(np.int32), y.view(np.int32)), (start, layer)
    new.close(), old.close()


@pytest.mark.parametrize("options", [dict(draft_len=4), dict(draft_len=0), dict(draft_len=15), dict(draft_len=3, use_graphs=False), dict(draft_len=4, refresh=True),
                                     dict(draft_len=4, exit_mode=1, gamma0=0.0011), dict(draft_len=4, temperature=0.8, seed=3), dict(draft_len=0, temperature=0.8, seed=3)],
                         ids=lambda o: "-".join(f"{k}{v}" for k, v in o.items()))
def test_loops_emit_the_same(options):
    """The drafts' ends left to the next pass's first launch, in every form of the loop; the cache crosses a group of 256 keys and the end of these
    kernels' contexts (where a cycle goes back to one launch per step)."""
    s = si.SHAPES["tiny"]
    new, old = engines(s)
    rng = np.random.default_rng(4)
    for n_prompt, n_new in ((9, 40), (241, 32), (745, 40)):
        prompt = rng.integers(0, s.vocab, n_prompt, dtype=np.int32)
        for masked in (dict(alpha=0.985, m=2, n=1), dict(fixed_mask=np.array([1, 0, 0, 1, 1, 1, 0, 0], np.uint8))):
            if "refresh" in options and "fixed_mask" in masked:
                continue
            (ta, sa, ma), (tb, sb, mb) = (e.generate(prompt, n_new, **options, **masked) for e in (new, old))
            assert np.array_equal(ta, tb) and np.array_equal(ma, mb), (n_prompt, masked)
            assert all(sa[k] == sb[k] for k in ("cycles", "drafted", "accepted", "emitted", "mask_changes", "gamma"))
    new.close(), old.close()


@pytest.mark.parametrize("vocab", [1024, 40000])
@pytest.mark.parametrize("silent", [True, False], ids=["silent", "ordinary"])
def test_drafts_without_any_sublayer(vocab, silent):
    """A draft step under a mask that leaves out every sublayer is the LM head alone, a launch that needs the token of the step before and writes the next
    candidates.  40000 entries: more LM-head workgroups than run at once.  silent: the sublayers' output projections are zero, so the full model says what the
    draft model says and every draft of a greedy loop is kept, if each step took the token of the step before."""
    s = si.SHAPES["tiny"].with_(vocab=vocab)
    W = [(t, l, 0 * w if silent and t in (si.T_WO, si.T_WD) else w) for t, l, w in si.all_tensors(s, 5, gain_std=0.1)]
    new, old = (asd.Engine(asd.make_config(s, 128, page_tokens=64, debug_tune=t)).load(W) for t in (None, "small=0"))
    prompt = np.random.default_rng(6).integers(0, vocab, 12, dtype=np.int32)
    for options in (dict(draft_len=2), dict(draft_len=4), dict(draft_len=4, use_graphs=False), dict(draft_len=9), dict(draft_len=4, exit_mode=1),
                    dict(draft_len=4, temperature=0.8, seed=3)):
        for masked in (dict(fixed_mask=np.ones(2 * s.n_layers, np.uint8)), dict(alpha=0.985, m=1, n=0)):
            (ta, sa, ma), (tb, sb, mb) = (e.generate(prompt, 40, **options, **masked) for e in (new, old))
            assert ma.all() and mb.all(), (options, masked)
            assert np.array_equal(ta, tb), (options, masked)
            assert all(sa[k] == sb[k] for k in ("cycles", "drafted", "accepted", "emitted")), (options, masked)
            assert not silent or "temperature" in options or sa["accepted"] == sa["drafted"] > 0, (options, masked)
    new.close(), old.close()


def test_a_token_outside_the_vocabulary_is_reported():
    import torch
    s = si.SHAPES["tiny"]
    new, old = engines(s, 128)
    for e in (new, old):
        for ids in ([5, s.vocab, 7], [-1]):
            t = torch.tensor(ids, dtype=torch.int32, device="cuda:0")
            lg = torch.zeros((len(ids), s.vocab), device="cuda:0")
            torch.cuda.synchronize()
            e.forward_noalloc(t, 0, commit=False, d_logits=lg)
            with pytest.raises(asd.AsdError):
                e.check()
        t = torch.tensor([5], dtype=torch.int32, device="cuda:0")
        torch.cuda.synchronize()
        e.forward_noalloc(t, 0, commit=False)
        e.check()
    new.close(), old.close()


def test_the_profiled_pass_is_the_pass_that_runs():
    """One launch per kept sublayer, the LM head and the finish, with the bytes of all steps; the launches of one launch per step where that is what runs."""
    s = si.SHAPES["tiny"]
    new, old = engines(s, 128)
    skip = np.array([1, 0, 0, 1, 1, 1, 0, 0], np.uint8)
    for e in (new, old):
        e.prefill(np.arange(20, dtype=np.int32))
    for rows, mask in ((1, None), (5, skip), (8, np.ones(8, np.uint8)), (9, skip)):
        a, b = (e.profile_forward(rows, mask) for e in (new, old))
        kept = np.zeros(8, np.uint8) if mask is None else mask
        launches = {k: v["launches"] for k, v in a.items() if k != "ms_total" and v["launches"]}
        att, mlp = int((kept[0::2] == 0).sum()), int((kept[1::2] == 0).sum())
        want = dict(attn=att, gateup=mlp, lmhead=1, finish=1) if rows <= 8 else dict(embed=1, qkv=att, attn=att, oproj=att, gateup=mlp, down=mlp, lmhead=1, finish=1)
        assert launches == {k: v for k, v in want.items() if v}, rows
        total = lambda p: sum(v["bytes"] for k, v in p.items() if k != "ms_total")
        assert abs(total(a) - total(b)) <= 1e-12 * total(b) and total(b) == pytest.approx(e.time_pass(rows, mask, 1)[1], rel=1e-12), rows
    new.close(), old.close()
