"""The ring kernel of the prompt GEMMs, every shape: blocks of one row block (whose weights are read past the caches) and of several,
with partly filled last tiles, chunks and quads of rows, K ranges shorter than the ring and odd ones, against the four-wave kernel: the same bits,
because every output is one wave's sum over its K slice in k-block order in both."""
import numpy as np
import pytest

import asd_inputs as si
import paper_2410_01028_amd as asd

pytestmark = pytest.mark.gpu

OTHER = "pf_qkv=4,1,2;pf_o=4,4,2;pf_gu=4,1,2;pf_down=4,4,2"
# 24 QKV tiles, 14 residual tiles, 21 gate/up pairs, 7, 6 and 11 k-blocks; 40 QKV tiles, 32 residual tiles, 35 pairs, 16, 16 and 18 k-blocks (bf16), twice those in fp32
RAGGED = si.Shape("ragged", 2, 224, 6, 3, 32, 336, 320, si.DT_BF16, 8, 8, 2)
WIDER = si.Shape("wider", 2, 512, 6, 2, 64, 560, 320, si.DT_BF16, 8, 8, 2)


def run(shape, n, tune, W):
    eng = asd.Engine(asd.make_config(shape, n + 80, debug_tune=tune)).load(W)
    eng.set_page_table(np.random.default_rng(n).permutation(-(-(n + 80) // 64)))
    out = (*eng.prefill(si.prompt(n, n, shape.vocab), want_logits=True), *eng.get_kv(0, 0, n + 16), *eng.get_kv(1, 0, n + 16))
    eng.close()
    return out


@pytest.mark.parametrize("shape", [RAGGED, WIDER, WIDER.with_(dtype=si.DT_F32)], ids=lambda s: f"{s.name}-{s.dtype}")
@pytest.mark.parametrize("n", [17, 35, 66, 161, 322])
def test_every_ring_shape_gives_the_bits_of_the_four_wave_kernel(shape, n):
    W = list(si.all_tensors(shape, 4, 0.1))
    want = run(shape, n, OTHER, W)
    assert not want[3][n:].any() and not want[4][n:].any()                 # nothing behind the prompt
    for v in range(16):
        tune = f"pf_ring={v},4"
        assert set(asd.plan_prompt(asd.make_config(shape, n + 80, debug_tune=tune), n)[0]["tile"].values()) == {v}
        got = run(shape, n, tune, W)
        assert all(np.array_equal(a, b) for a, b in zip(want, got)), v
