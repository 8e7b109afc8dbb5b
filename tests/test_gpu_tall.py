"""GPU parity of the tall product tiles (128 rows x 256 columns over blocked
weights, taken by products of many rows): single products, prefills, batched
steps and the head against the oracle, bit for bit, at sizes that fill no
tile, no stage of words and no byte of the value cache.  Every test states
which of its products take the tall tiles."""
import numpy as np
import pytest

from oracle import nmdlm_oracle as O
from workloads import synth

from ._gpu import assert_same, need_gpu, padding_bits_zero, run_qbsm
from ._plan import CUR, HEAD, plan, step_plans
from .test_gpu_batch import _batched_matches_independent
from .test_gpu_block import _check_block

pytestmark = pytest.mark.gpu


def tall(plans):
    return {k for k, p in plans.items() if p.kernel == "tall"}


# T, M, K, N, spikes alone on tall tiles, currents alone on tall tiles: enough
# workgroups or tiles, or just too few (currents: 448 tiles of 64 columns at K <= 1024).
# N of every remainder by four: rows of currents at every alignment, the last store
# of 1, 2, 3 and 4 of them
PRODUCTS = [
    (4, 879, 500, 1000, True, True),     # 28 row blocks, the last of 15 tokens; the last tile of 40 columns
    (4, 897, 65, 1030, True, True),      # two words of K; one token in the last row block; tiles past N
    (8, 440, 257, 1024, True, True),     # five words (a stage and one more), 8 of 16 tokens
    (2, 1740, 512, 1024, True, True),    # 64-token row blocks, the last of 12
    (1, 3470, 320, 1000, True, True),    # 128-token row blocks, the last of 14
    (4, 1270, 1000, 1000, True, True),   # 16 words, 160 workgroups
    (4, 512, 2100, 2500, True, True),    # 33 words, 160 workgroups
    (4, 879, 257, 1001, True, True),
    (1, 3470, 65, 1003, True, True),
    (4, 889, 1000, 1000, False, True),   # 112 workgroups: spikes on lean tiles
    (2, 890, 700, 2047, False, True),
    (8, 1000, 64, 449, True, True),      # 126 workgroups: four of the last group's columns
    (4, 4000, 100, 193, True, True),     # 125, the last column alone in its tile
    (4, 860, 500, 950, False, False),    # 405 tiles: the other kernels
    (4, 379, 500, 1000, False, False),
    (1, 1530, 320, 1000, False, False),
    (2, 760, 512, 1024, False, False),
    (8, 190, 257, 1024, False, False),
    (4, 350, 512, 1000, False, False),
    (8, 1780, 257, 70, True, False),     # 112 workgroups, but two column tiles in each
]


@pytest.mark.parametrize("shape", PRODUCTS, ids=["T%dM%dK%dN%d" % s[:4] for s in PRODUCTS])
@pytest.mark.parametrize("flags", [0, 1], ids=["skip", "dense"])
def test_products(shape, flags):
    need_gpu()
    T, M, K, N, spikes_tall, currents_tall = shape
    assert (plan(T, M, K, N, blocked=1, flags=flags).kernel == "tall") == spikes_tall
    assert (plan(T, M, K, N, mode=CUR, blocked=1, bias=1, cur=1, flags=flags).kernel == "tall") == currents_tall
    c = synth.make_qbsm_case(7 + K + N, T, M, K, N, 0.06, bias_range=0)
    I = O.qbsm(c.S, c.W, c.bias)
    _, spk, st, words, _ = run_qbsm(c.S, c.W, theta=c.theta, want_cur=False, blocked=True, flags=flags)
    assert_same(spk, O.if_neuron(I, c.theta)[0])
    assert padding_bits_zero(words, N)
    assert st["k_active"] == (K if flags else O.active_rows(c.S).size)
    bias = np.arange(N, dtype=np.int32) - 50
    cur, _, _, _, _ = run_qbsm(c.S, c.W, bias=bias, blocked=True, flags=flags)   # currents alone
    assert_same(cur, I + bias)


@pytest.mark.parametrize("theta", [1, 1 << 26, (1 << 26) + 1, 2 ** 31 - 1])
def test_thresholds_at_the_32_bit_bound(theta):
    """Full spikes against weights of one sign: the largest and smallest
    membranes, with thresholds on either side of the 32-bit epilogue's bound."""
    need_gpu()
    T, M, K, N = 8, 480, 512, 1024
    assert plan(T, M, K, N, theta=theta, blocked=1).kernel == ("tall" if theta <= 1 << 26 else "lean")
    S = np.ones((T, M, K), dtype=bool)
    W = np.full((K, N), 127, dtype=np.int8)
    W[:, ::2] = -127
    _, spk, _, _, _ = run_qbsm(S, W, theta=theta, want_cur=False, blocked=True)
    assert_same(spk, O.if_neuron(O.qbsm(S, W, np.zeros(N, np.int32)), theta)[0])


@pytest.mark.parametrize("C,M,d,H,F,T", [
    (1192, 1, 256, 4, 800, 4),    # 38 row blocks, the last of 8 tokens
    (1189, 3, 256, 2, 1040, 4),   # the last row block's tokens end within a byte of the value cache
    (598, 5, 256, 4, 784, 8),     # 16-token row blocks, the last of 6
    (3, 1190, 256, 4, 800, 4),    # the block itself, from position 3 on: bits set with atomics
])
def test_prefill_and_step(C, M, d, H, F, T):
    need_gpu()
    R, pos0 = max((C, 0), (M, C))
    assert tall(step_plans(T, R, d, F, pos0)) == {"qkv", "up"}
    _check_block(synth.block_case(seed=C, C=C, M=M, d=d, H=H, F=F, T=T), blocked=True)


EVERY = {"qkv", "o", "up", "dn"}


@pytest.mark.parametrize("n,C,M,d,H,F,T,on_tall", [
    (128, 16, 16, 512, 8, 512, 4, EVERY),   # two sequences a row block, whole bytes
    (110, 24, 20, 512, 8, 512, 4, EVERY),   # sequences straddle the row blocks, runs of 4 to 20 tokens
    (100, 12, 12, 512, 4, 512, 4, {"qkv"}),  # the same from position 12 on
    (100, 12, 10, 512, 8, 512, 8, EVERY),   # 16-token row blocks over 10-token sequences
    (113, 8, 32, 512, 8, 496, 2, EVERY - {"qkv"}),  # 64-token row blocks (too long for the value cache)
    (57, 16, 128, 512, 4, 512, 1, EVERY - {"qkv"}),  # 128-token row blocks
])
def test_batched_step(n, C, M, d, H, F, T, on_tall):
    need_gpu()
    assert tall(step_plans(T, M, d, F, C, n)) == on_tall
    _batched_matches_independent(n, C, M, d, H, F, 0, T, blocked=True)


@pytest.mark.parametrize("M,V,kernel", [(310, 3008, "tall"), (310, 2992, "tall"), (157, 3008, "lean"),
                                        (16, 3008, "lean")])
def test_head_logits(M, V, kernel):
    """10 row blocks x 12 column groups, the last of 22 tokens and three column
    tiles, the last of 64 or 48 columns; and the same head on lean tiles."""
    torch, B = need_gpu()
    m = synth.make_mdlm(5, 1, d=256, H=4, F=256, V=V, T=4, max_pos=320)
    assert plan(4, M, m.d, m.V, mode=HEAD, blocked=1).kernel == kernel
    toks = synth.random_tokens(6, M, m.V).astype(np.int32)
    dm = B.DeviceModel.from_mdlm(m, M, blocked=True)
    ws = B.workspace(B.nmdlm_block_step_workspace_size(dm, M, 0))
    y = torch.empty((4, M, 4), dtype=torch.int64, device="cuda")
    logits = torch.empty((M, m.V), dtype=torch.float32, device="cuda")
    masked = torch.ones(M, dtype=torch.uint8, device="cuda")
    B.nmdlm_block_step(dm, B.step_io(M, 0, tokens=torch.from_numpy(toks).cuda(), masked=masked,
                                     k_unmask=1, y_out=y, logits=logits), ws)
    torch.cuda.synchronize()
    Y = synth.unpack_bits(B.from_dev_bits(y), m.d)
    acc = Y.sum(0).astype(np.int64) @ m.W_head.astype(np.int64)
    want = acc.astype(np.float32) * m.scale    # one float32 product per entry: the same bits
    assert np.array_equal(logits.cpu().numpy(), want)
