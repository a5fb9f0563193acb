"""The end of a prompt taken in blocks: the last row on its way to the LM head, the last block's cosine sums, and the results in host memory.

Lengths: the shortest prompt in blocks, a whole and a begun 16-row chunk, and a last block of a single row.
"""
import numpy as np
import pytest

import asd_inputs as si
import paper_2410_01028_amd as asd
from test_gpu_parity import BF_GQA, COS_TOL, TOL, build_pair, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [si.SHAPES["tiny"], BF_GQA], ids=lambda s: s.name)
@pytest.mark.parametrize("n", [17, 32, 33, 513])
def test_last_row_sums_and_results(shape, n):
    eng, orc = build_pair(shape, seed=6, max_seq=n + 8)
    if n == 513:
        assert asd.plan_prompt(eng.cfg, n)[-1]["rows"] == 1
    toks = si.prompt(7, n, shape.vocab)
    o = orc.forward(toks, 0)
    other = si.prompt(8, n, shape.vocab)
    eng.prefill(other, want_logits=True)                    # other results in the host's memory
    first, acs, lg = eng.prefill(toks, want_logits=True)
    assert first == int(np.argmax(lg))
    assert rel_err(lg, o["logits"][-1]) < TOL[shape.dtype]
    assert np.abs(acs - o["cos"]).max() < COS_TOL
    eng.prefill(other)
    again, acs2 = eng.prefill(toks)[:2]
    assert again == first and np.array_equal(acs, acs2)


def test_last_row_without_a_maximum_is_reported():
    s = si.SHAPES["tiny"]
    W = [(t, l, np.full_like(w, np.nan) if t == si.T_FINAL_NORM else w) for t, l, w in si.all_tensors(s, 3)]
    eng = asd.Engine(asd.make_config(s, 128)).load(W)
    with pytest.raises(asd.AsdError, match="finite maximum"):
        eng.prefill(si.prompt(1, 40, s.vocab))
