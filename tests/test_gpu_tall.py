"""GPU parity of the tall product tiles (128 rows x 256 columns over blocked
weights, taken by products of many rows): single products, prefills, batched
steps and the head against the oracle, bit for bit, at sizes that fill no
tile, no stage of words and no byte of the value cache."""
import numpy as np
import pytest

from oracle import nmdlm_oracle as O
from workloads import synth

from ._gpu import assert_same, need_gpu, padding_bits_zero, run_qbsm
from .test_gpu_batch import _batched_matches_independent
from .test_gpu_block import _check_block

pytestmark = pytest.mark.gpu

PRODUCTS = [  # T, M, K, N: enough workgroups for the tall tiles, or just too few
    (4, 379, 500, 1000),     # 12 row blocks, the last of 27 tokens; the last tile of 40 columns
    (4, 385, 65, 1030),      # two words of K; one token in the last row block; tiles past N
    (8, 190, 257, 1024),     # five words (a stage and one more), 14 of 16 tokens
    (2, 760, 512, 1024),     # 64-token row blocks
    (1, 1530, 320, 1000),    # 128-token row blocks
    (4, 896, 1000, 1000),    # 16 words, 112 workgroups
    (4, 512, 2100, 2500),    # 33 words, 160 workgroups
    (4, 350, 512, 1000),     # 44 workgroups: the other kernels
]


@pytest.mark.parametrize("shape", PRODUCTS, ids=["T%dM%dK%dN%d" % s for s in PRODUCTS])
@pytest.mark.parametrize("flags", [0, 1], ids=["skip", "dense"])
def test_products(shape, flags):
    need_gpu()
    T, M, K, N = shape
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
    T, M, K, N = 8, 190, 512, 1024
    S = np.ones((T, M, K), dtype=bool)
    W = np.full((K, N), 127, dtype=np.int8)
    W[:, ::2] = -127
    _, spk, _, _, _ = run_qbsm(S, W, theta=theta, want_cur=False, blocked=True)
    assert_same(spk, O.if_neuron(O.qbsm(S, W, np.zeros(N, np.int32)), theta)[0])


@pytest.mark.parametrize("C,M,d,H,F,T", [
    (520, 1, 256, 4, 800, 4),     # prefill of 520: 17 row blocks x 3 column groups, the last of 8 tokens
    (517, 3, 256, 2, 1040, 4),    # the last row block's tokens end within a byte of the value cache
    (262, 5, 256, 4, 784, 8),     # 16-token row blocks
])
def test_prefill_and_step(C, M, d, H, F, T):
    need_gpu()
    _check_block(synth.block_case(seed=C, C=C, M=M, d=d, H=H, F=F, T=T), blocked=True)


@pytest.mark.parametrize("n,C,M,d,H,F,T", [
    (36, 16, 16, 256, 4, 512, 4),   # two sequences a row block, whole bytes
    (30, 24, 20, 256, 4, 512, 4),   # sequences straddle the row blocks, runs of 4 to 20 tokens
    (56, 12, 10, 256, 4, 512, 8),   # 16-token row blocks over 10-token sequences
])
def test_batched_step(n, C, M, d, H, F, T):
    _batched_matches_independent(n, C, M, d, H, F, 0, T, blocked=True)


def test_head_logits():
    torch, B = need_gpu()
    m = synth.make_mdlm(5, 1, d=256, H=4, F=256, V=3008, T=4, max_pos=160)
    M = 157                                    # 5 row blocks x 12 column groups
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
