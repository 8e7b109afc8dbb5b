"""GPU parity of the lean product (blocked weights of few rows, every word
read, weights in flight before the spikes): spikes and statistics against the
oracle at the edges of its tiles, of its groups of words and of its staging
batches; and the block steps that run on it alone (residual, table, unions,
value cache).  Every test states that its products take it."""
import numpy as np
import pytest

from oracle import nmdlm_oracle as O
from workloads import synth

from ._gpu import assert_same, need_gpu, padding_bits_zero, run_qbsm
from ._plan import plan, step_plans
from .test_gpu_batch import _batched_matches_independent
from .test_gpu_block import _check_block

pytestmark = pytest.mark.gpu

SHAPES = [  # T, M, K, N, rows and waves of a tile
    (1, 1, 1, 1, 16, 8),            # one row, one word, one column
    (4, 1, 65, 63, 16, 8),
    (3, 5, 200, 130, 16, 8),        # T that divides no tile height
    (5, 7, 2048, 70, 16, 8),        # 32 words: four per wave of eight
    (8, 2, 2049, 64, 16, 16),       # 33 words: sixteen waves, three words at most
    (8, 9, 4000, 200, 16, 16),      # 63 words
    (2, 30, 4160, 100, 16, 16),     # 65 words: a second group for wave 0 only
    (4, 13, 8200, 300, 16, 16),     # 129 words, a partial staging batch
    (4, 9, 16300, 130, 16, 16),     # 255 words: eight staging batches
    (4, 20, 20000, 900, 16, 16),    # 75 tiles of a K that few tiles would split
    (4, 65, 40000, 70, 16, 16),     # 625 words: most of a CU's LDS
    (1, 256, 65536, 64, 16, 16),
    (4, 32, 1000, 6200, 64, 8),     # two row groups or four, 97 column tiles
    (4, 31, 2100, 8200, 64, 4),     # 129 column tiles, the last row block ragged
    (8, 24, 130, 16500, 64, 4),     # 64-row tiles of four waves, three words
    (4, 48, 300, 20000, 64, 4),
    (4, 60, 5000, 4100, 64, 8),     # 64-row tiles of eight waves, K over two staging batches
    (1, 65, 700, 900, 16, 8),       # one step: a row is a token
    (8, 17, 7600, 5700, 32, 8),     # 32-row tiles of a long K, the last row block of one token
]


@pytest.mark.parametrize("shape", SHAPES, ids=["T%dM%dK%dN%d" % s[:4] for s in SHAPES])
def test_products(shape):
    need_gpu()
    T, M, K, N, rows, waves = shape
    p = plan(T, M, K, N, blocked=1)
    assert (p.kernel, p.rows, p.waves) == ("lean", rows, waves)
    for seed, density, flags in ((1, 0.15, 0), (2, 0.004, 0), (3, 0.3, 1)):
        c = synth.make_qbsm_case(seed + K + N, T, M, K, N, density, bias_range=0)
        _, spk, st, words, _ = run_qbsm(c.S, c.W, theta=c.theta, want_cur=False, blocked=True,
                                        flags=flags)
        assert_same(spk, O.if_neuron(O.qbsm(c.S, c.W, c.bias), c.theta)[0], f"density {density}")
        assert padding_bits_zero(words, N)
        k_act = K if flags else O.active_rows(c.S).size
        assert (st["k_total"], st["k_active"], st["n"], st["weight_bytes"]) == (K, k_act, N, k_act * N)


def test_silent_block():
    need_gpu()
    S = np.zeros((4, 8, 500), dtype=bool)
    W = synth.int8_uniform(synth.stream(1, 1), (500, 300))
    _, spk, st, _, _ = run_qbsm(S, W, theta=1, want_cur=False, blocked=True)
    assert not spk.any() and st["k_active"] == 0


@pytest.mark.parametrize("C,M,d,H,F,T", [
    (40, 16, 256, 4, 800, 4),      # 64 rows, the value cache in bytes; the context in 160 rows
    (45, 17, 256, 2, 1040, 4),     # one token past a tile, bits of the value cache set with atomics
    (61, 5, 512, 4, 528, 3),       # five tokens a row block, across a word of the value cache
    (30, 9, 256, 4, 784, 8),
    (70, 65, 128, 2, 256, 1),
    (16, 32, 2048, 16, 8192, 4),   # the 12-layer model's layer: 64-row tiles of eight waves, 16-row ones of sixteen
])
def test_block_step(C, M, d, H, F, T):
    need_gpu()
    for rows, pos0 in ((C, 0), (M, C)):
        assert {p.kernel for p in step_plans(T, rows, d, F, pos0).values()} == {"lean"}
    _check_block(synth.block_case(seed=C, C=C, M=M, d=d, H=H, F=F, T=T), blocked=True)


@pytest.mark.parametrize("n,C,M,d,H,F,T", [
    (5, 24, 12, 256, 4, 512, 4),    # 12-token sequences: four tokens a row block of the value cache
    (6, 32, 16, 512, 8, 512, 8),    # (d = 256 runs QKV on the word kernel: 1152 tiles of four words)
])
def test_batched_step(n, C, M, d, H, F, T):
    need_gpu()
    assert {p.kernel for p in step_plans(T, M, d, F, C, n).values()} == {"lean"}
    _batched_matches_independent(n, C, M, d, H, F, 0, T, blocked=True)
