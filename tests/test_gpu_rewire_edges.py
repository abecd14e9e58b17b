"""GPU parity of haste_rewire at the edges of its chunks and of its ties, against the CPU oracle (exact).

A wave moves whole label rows in chunks of up to 1024 (small groups: 256) values and 64 rows, in accesses of 16, 4 or 2
bytes by what divides a row; a key equal to the threshold is pruned if few enough equal ones precede
it, counted from the start of its 1024-key block.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import say
from test_gpu_rewire import BF16, F32, _run, hs, orc  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # name, K, G, F, H, dtype, rho, with velocity, levels (0: distinct weights; n: n magnitudes only)
    ("bf16_rows_past_64", 90, 150, 3, 40, BF16, 0.4, True, 0),
    ("bf16_one_slot", 700, 130, 1, 9, BF16, 0.3, True, 0),
    ("bf16_odd_chunks", 211, 37, 57, 300, BF16, 0.1, True, 0),
    ("bf16_even_rows", 130, 33, 62, 700, BF16, 0.2, True, 0),
    ("bf16_last_chunk_one_row", 100, 17, 64, 768, BF16, 0.1, True, 0),
    ("f32_odd", 90, 19, 129, 640, F32, 0.2, True, 0),
    ("f32_vec_remainder", 77, 41, 36, 512, F32, 0.15, True, 0),
    ("bf16_all_tied", 331, 4, 24, 256, BF16, 0.37, True, 1),
    ("bf16_ties_over_blocks", 257, 2, 200, 400, BF16, 0.45, False, 2),
    ("f32_ties", 1500, 1, 33, 128, F32, 0.31, True, 3),
    # groups of up to 256 weights (the smaller chunk), by access and 64-slot words, and one past it
    ("bf16_small", 900, 4, 64, 300, BF16, 0.2, True, 0),
    ("bf16_small_even", 700, 3, 30, 90, BF16, 0.3, True, 0),
    ("bf16_small_one", 2000, 1, 1, 9, BF16, 0.3, True, 0),
    ("bf16_small_odd", 1000, 2, 5, 64, BF16, 0.4, True, 0),
    ("bf16_small_two_words", 300, 2, 128, 600, BF16, 0.1, True, 0),
    ("bf16_small_four_words_odd", 300, 1, 255, 700, BF16, 0.2, True, 0),
    ("bf16_one_past", 60, 257, 1, 30, BF16, 0.3, True, 0),
    ("f32_small", 500, 4, 64, 256, F32, 0.2, True, 0),
    ("f32_small_two_words_odd", 400, 3, 77, 200, F32, 0.3, False, 0),
    ("f32_small_four_words", 200, 1, 256, 900, F32, 0.1, True, 0),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_rewire_edges_exact(hs, orc, case):  # noqa: F811
    name, K, G, F, H, dt, rho, with_m, levels = case
    say(f"[rewire edge] {name}: K={K} G={G} F={F} H={H} rho={rho}")
    rng = np.random.default_rng(K * F + G)
    idx = np.stack([np.sort(rng.choice(H, F, replace=False)) for _ in range(K)]).astype(np.int32)
    W = (rng.standard_normal((K * G, F)) / np.sqrt(F)).astype(np.float32)
    if levels:
        W = np.repeat(rng.integers(0, levels, (K, 1, F)), G, 1).reshape(K * G, F).astype(np.float32) * 0.25
    W = synth.bf16_bits(W) if dt == BF16 else W
    m = rng.standard_normal((K * G, F)).astype(np.float32) if with_m else None
    seed = 1234567 + F
    got_n, gi, gW, gm = _run(hs, K, G, F, H, dt, idx, W, m, rho, 1, seed)
    wi, wW, wm, n, _ = orc.rewire(idx, W, m, G, H, dt, rho, True, seed)
    assert got_n == n
    np.testing.assert_array_equal(gi, wi)
    np.testing.assert_array_equal(gW, wW)
    if with_m:
        np.testing.assert_array_equal(gm, wm)
