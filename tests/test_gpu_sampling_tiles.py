"""The sampling kernels at vocabulary sizes around their 256-value tiles and 16-wave split, and at both ends of the register
variant, against the oracle's rule on identical logits (draws within MARGIN of a threshold are left out: either outcome is
right there), and the two variants against each other draw for draw."""
import numpy as np
import pytest

import asd_inputs as si
import paper_2410_01028_amd as asd
from test_gpu_sampling import MARGIN, oracle_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [16, 256, 272, 4080, 4112, 32768, 32784])
def test_draws_at_the_edges_of_the_tiles(V):
    shape = si.Shape("v", 1, 64, 2, 2, 32, 64, V, si.DT_F32, 4, 4, 2)
    engines = [asd.Engine(asd.make_config(shape, 64, debug_flags=f)) for f in (0, asd.DBG_SAMPLE_MEM)]
    rng = np.random.default_rng(V)
    compared = 0
    for trial in range(24):
        kk = int(rng.integers(0, 6))
        p = rng.normal(0, 2.0, (kk + 1, V)).astype(np.float32)
        q = (p[:kk] + rng.normal(0, float(rng.choice([0.1, 1.0])), (kk, V))).astype(np.float32)
        if trial % 4 == 3:                    # all weight in the last / first few values, the rest far below
            p -= 200.0
            p[:, -3:] += 200.0
            q[:, :2] += 300.0
        seed, index0 = int(rng.integers(0, 2 ** 40)), int(rng.integers(0, 1000))
        got = [e.spec_sample(q, p, 0.8, seed, index0) for e in engines]
        assert np.array_equal(got[0][0], got[1][0]) and got[0][1:] == got[1][1:]
        wd, wa, wn, mg = oracle_step(q.astype(np.float64), p.astype(np.float64), 0.8, seed, index0)
        if mg >= MARGIN:
            compared += 1
            assert np.array_equal(got[0][0], wd) and got[0][1] == wa and got[0][2] == wn, (trial, kk, mg)
    assert compared >= 12
    for e in engines:
        e.close()


@pytest.mark.parametrize("drafts", [0, 3])
def test_sampled_decoding_reports_rows_without_a_maximum(drafts):
    """Sampled passes run without the greedy finish: the sampling kernels report such rows in its place."""
    s = si.SHAPES["tiny"]
    eng = asd.Engine(asd.make_config(s, 128))
    eng.init_synthetic(0)
    first = eng.prefill([1, 2, 3, 4])[0]
    kw = dict(temperature=0.8, seed=1, fixed_mask=np.zeros(2 * s.n_layers, np.uint8))
    eng.decode(first, 4, drafts, **kw)
    eng.set_weight(si.T_FINAL_NORM, 0, np.full(s.d_model, np.nan, np.float32))
    with pytest.raises(asd.AsdError) as ei:
        eng.decode(first, 4, drafts, **kw)
    assert ei.value.code == asd.E_STATE
    eng.close()


@pytest.mark.parametrize("V", [16, 272, 32768, 32784])
def test_rows_with_nan_draw_their_last_positive_weight(V):
    """A row with a NaN has no running sum: draft draws, extra draws and replacements then take the last index with a positive
    weight (masked -inf logits have none), in both variants of the kernels."""
    shape = si.Shape("v", 1, 64, 2, 2, 32, 64, V, si.DT_F32, 4, 4, 2)
    rng = np.random.default_rng(V)
    p = rng.normal(0, 2.0, (3, V)).astype(np.float32)
    q = p[:2] + rng.normal(0, 0.5, (2, V)).astype(np.float32)
    clean = p[2:].copy()
    for rows in (p, q):
        rows[:, V // 3] = np.nan
        rows[:, V - 2:] = -np.inf
    q[1, V - 5:] = -np.inf
    for flags in (0, asd.DBG_SAMPLE_MEM):
        eng = asd.Engine(asd.make_config(shape, 64, debug_flags=flags))
        drafts, acc, nxt = eng.spec_sample(q, p, 0.8, 5, 0)
        assert list(drafts) == [V - 3, V - 6] and acc == 0 and nxt == V - 3      # a NaN ratio keeps no draft
        assert eng.spec_sample(np.zeros((0, V), np.float32), p[:1], 0.8, 5, 0)[2] == V - 3
        assert eng.spec_sample(np.zeros((0, V), np.float32), np.full((1, V), np.nan, np.float32), 0.8, 5, 0)[2] == 0
        masked = clean.copy()
        masked[:, 3:] = -np.inf                                                   # ordinary masked rows: only what is left
        assert all(eng.spec_sample(np.zeros((0, V), np.float32), masked, 0.8, s, 0)[2] < 3 for s in range(20))
        eng.close()


@pytest.mark.parametrize("flags", [0, asd.DBG_SAMPLE_MEM], ids=["registers", "memory"])
@pytest.mark.parametrize("dtype", [si.DT_BF16, si.DT_F32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("drafts", [1, 2, 5])
def test_the_drawn_token_is_the_next_draft_steps_input(dtype, drafts, flags):
    """A draw between two draft steps embeds its token itself.  Drafts of the whole model are its own draws: the same bits in the
    draft step and the verification, hence all kept, unless a step had another token's embedding."""
    s = si.Shape("d", 2, 272, 2, 1, 64, 304, 1040, dtype, 4, 4, 2)
    eng = asd.Engine(asd.make_config(s, 192, debug_flags=flags, debug_tune="small=0"))
    eng.init_synthetic(5)
    first = eng.prefill(si.prompt(2, 40, s.vocab))[0]
    kw = dict(temperature=0.9, seed=11, fixed_mask=np.zeros(2 * s.n_layers, np.uint8))
    got = []
    for graphs in (False, True):
        eng.reset()
        assert eng.prefill(si.prompt(2, 40, s.vocab))[0] == first
        toks, st, _ = eng.decode(first, 24, drafts, use_graphs=graphs, **kw)
        assert st["accepted"] == st["drafted"] > 0
        got.append(toks)
    assert np.array_equal(got[0], got[1])
    eng.close()
