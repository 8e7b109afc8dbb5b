"""GPU parity of the lean product (blocked weights of few rows, every word
read, weights in flight before the spikes): spikes and statistics against the
oracle at the edges of its tiles, of its groups of words and of its staging
batches."""
import numpy as np
import pytest

from oracle import nmdlm_oracle as O
from workloads import synth

from ._gpu import assert_same, need_gpu, padding_bits_zero, run_qbsm

pytestmark = pytest.mark.gpu

SHAPES = [  # T, M, K, N
    (1, 1, 1, 1),            # one row, one word, one column
    (4, 1, 65, 63),
    (3, 5, 200, 130),        # T that divides no tile height
    (5, 7, 2048, 70),        # 32 words: four per wave of eight
    (8, 2, 2049, 64),        # 33 words: sixteen waves, three words at most
    (8, 9, 4000, 200),       # 63 words
    (2, 30, 4160, 100),      # 65 words: a second group for wave 0 only
    (4, 13, 8200, 300),      # 129 words, a partial staging batch
    (4, 32, 1000, 6200),     # two row groups or four, 97 column tiles
    (4, 31, 2100, 8200),     # 64-row tiles of eight waves, the last row block ragged
    (8, 24, 130, 16500),     # 64-row tiles, three words
    (4, 48, 300, 20000),     # 64-row tiles of four waves
    (4, 60, 5000, 4100),     # 64-row tiles, K over two staging batches
    (1, 65, 700, 900),       # one step: a row is a token
]


@pytest.mark.parametrize("shape", SHAPES, ids=["T%dM%dK%dN%d" % s for s in SHAPES])
def test_products(shape):
    need_gpu()
    T, M, K, N = shape
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
