"""Where a prompt block's activations lie: over the staging region of weight uploads, with an odd number of KiB from chunk to chunk where
that fits and without where not.  Long blocks in every tile shape of the ring kernel, on both strides, with K ranges that take a 16-stage ring
round more than twice, give the bits of the four-wave kernel; 512 rows over the staging region leave weights and results alone."""
import numpy as np
import pytest

import asd_inputs as si
import paper_2410_01028_amd as asd

pytestmark = pytest.mark.gpu

# 204 QKV tiles, 68 residual tiles, 76 gate/up pairs; 34, 34 and 38 k-blocks, no padding
DEEP = si.Shape("deep", 1, 1088, 17, 17, 64, 1216, 320, si.DT_BF16, 8, 8, 2)
FOUR_WAVE = "pf_qkv=4,1,2;pf_o=4,1,2;pf_gu=4,1,2;pf_down=4,1,2"


def workspace(s, rows, odd):
    """Bytes of a block's workspace (64-byte multiples aside): residual rows, partial sums, three row arrays, four activations."""
    kb = [-(-k // 32) | odd for k in (s.d_model, s.q_dim, s.q_dim, s.d_ffn)]
    return 4 * rows * s.d_model + 4 * 4096 * s.d_model + 4 * rows * (2 + 2 * s.n_layers) + rows // 16 * sum(kb) * 2048


def with_staging(s, least, below):
    """The shape with a vocabulary in the middle of those whose staging region (the embedding's bytes + 4 KiB) takes [least, below) bytes more than 512 rows do."""
    own = workspace(s, 512, 0)
    vocab = ((least + below) // 2 - own - 4096) // (2 * s.d_model) // 16 * 16
    assert least - own + 8192 < 2 * vocab * s.d_model + 4096 < below - own - 8192
    return s.with_(vocab=vocab)


ROWS_1024 = with_staging(DEEP, workspace(DEEP, 1024, 1), workspace(DEEP, 2048, 0))
ROWS_1024_EVEN = with_staging(DEEP, workspace(DEEP, 1024, 0), workspace(DEEP, 1024, 1))
ROWS_512_ODD = with_staging(DEEP, workspace(DEEP, 512, 1), workspace(DEEP, 1024, 0))


def run(shape, n, tune, W):
    cfg = asd.make_config(shape, n + 80, debug_tune=tune)
    plan = asd.plan_prompt(cfg, n)
    assert len(plan) == 1 and plan[0]["slices"]["oproj"] == plan[0]["slices"]["down"] == 1
    eng = asd.Engine(cfg).load(W)
    out = (*eng.prefill(si.prompt(n, n, shape.vocab), want_logits=True), *eng.get_kv(0, 0, n + 16))
    eng.close()
    return plan[0]["tile"], out


@pytest.mark.parametrize("shape", [ROWS_1024, ROWS_1024_EVEN], ids=["odd", "even"])
@pytest.mark.parametrize("n", [650, 1009])
def test_long_blocks_on_either_stride_give_the_bits_of_the_four_wave_kernel(shape, n):
    W = list(si.all_tensors(shape, 4, 0.1))
    tile, want = run(shape, n, FOUR_WAVE, W)
    assert set(tile.values()) == {-1}
    for v in range(16):
        tile, got = run(shape, n, f"pf_ring={v},1", W)
        assert set(tile.values()) == {v}
        assert all(np.array_equal(a, b) for a, b in zip(want, got)), v


def test_512_rows_over_the_staging_region_leave_weights_and_results_alone():
    shape, n = ROWS_512_ODD, 301
    assert max(b["rows"] for b in asd.plan_prompt(asd.make_config(shape, 2048), 2048)) == 512
    W = list(si.all_tensors(shape, 3))
    got = []
    for fill in (0x00, 0xFF):
        eng = asd.Engine(asd.make_config(shape, n + 16), arena_fill=fill).load(W)
        for _ in range(2):
            got.append((*eng.prefill(si.prompt(1, n, shape.vocab), want_logits=True), *eng.get_kv(0, 0, n)))
            for t, l, arr in W:
                assert np.array_equal(eng.get_weight(t, l, arr.shape, arr.dtype), arr)
        eng.close()
    for g in got[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(got[0], g))
