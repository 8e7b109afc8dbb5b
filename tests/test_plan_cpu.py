"""The choice of a product's kernel, on the host: bounds that a kernel needs."""
import os

import pytest

torch = pytest.importorskip("torch")
from paper_2607_24841_amd import binding as B  # noqa: E402

from ._plan import attn_route, plan, token_runs  # noqa: E402

pytestmark = pytest.mark.skipif(not os.path.exists(B.LIB_PATH), reason="libnmdlm.so not built")


@pytest.mark.parametrize("T,M,K,N", [(3, 1008, 64, 8 << 20), (3, 174000, 64, 33200), (5, 80, 64, 3 << 23),
                                     (7, 1000, 1, 3 << 20)])
def test_lean_grids_stay_below_the_float_quotient(T, M, K, N):
    """The lean product takes its tile's column as a float quotient, exact for
    fewer than 2^21 tiles (test_div_small); larger grids divide in integers."""
    p = plan(T, M, K, N, blocked=1)
    assert p.status == B.NMDLM_OK
    assert ((N + 63) // 64) * p.row_blocks >= 1 << 21
    assert p.kernel == "words"
    half = plan(T, M, K, N // 8, blocked=1)            # under the bound: lean again
    assert ((N // 8 + 63) // 64) * half.row_blocks < 1 << 21
    assert half.kernel == "lean"


@pytest.mark.parametrize("tokens", [16, 32])
@pytest.mark.parametrize("seq_len", [0, 4, 8, 10, 16, 20, 24, 33, 40, 72])
@pytest.mark.parametrize("pos0", [0, 4, 8, 13, 60, 64])
def test_channel_major_words_are_written_one_way(pos0, seq_len, tokens):
    """The runs of all row blocks cover every token once; no position word is
    written in bytes by one run and by atomics on the word by another, and no
    byte is stored by two."""
    M = 6 * seq_len if seq_len else 211
    seen, ways, owner = set(), {}, {}
    for y in range(-(-M // tokens)):
        m = y * tokens
        for i, (seq, pos, n, in_bytes) in enumerate(token_runs(pos0, seq_len, tokens, M, y)):
            assert n > 0
            for p in range(pos, pos + n):
                assert (seq, p) == ((m // seq_len, pos0 + m % seq_len) if seq_len else (0, pos0 + m))
                seen.add(m)
                m += 1
                ways.setdefault((seq, p // 64), set()).add(in_bytes)
                if in_bytes:
                    assert pos % 8 == 0
                    assert owner.setdefault((seq, p // 8), (y, i)) == (y, i)
    assert seen == set(range(M))
    assert all(len(w) == 1 for w in ways.values())


@pytest.mark.parametrize("T,M,K,N,kernel,splits", [
    (4, 4, 8192, 2048, "lean", 1),       # 32 tiles, 128 words: lean up to K = 10240
    (4, 4, 12000, 1024, "words", 4),     # 16 tiles of cold weights: a long K is split four ways
    (4, 4, 16384, 512, "lean", 1),       # 8 MB, in the last-level cache between uses
    (4, 4, 16385, 512, "words", 4),
    (4, 32, 20000, 512, "words", 4),     # 64 tiles
    (4, 33, 20000, 512, "lean", 1),      # 72 tiles: no split, lean again
    (4, 32, 34000, 512, "list", 1),      # beyond the word kernel's LDS: the active rows alone
    (4, 63, 34000, 70, "list", 1),
    (4, 64, 34000, 70, "lean", 1),       # 256 rows: most of the words are active
    (4, 15, 4096, 14336, "words", 1),    # fewer than 64 rows of a large matrix
    (4, 16, 4096, 14336, "lean", 1),
])
def test_lean_rule(T, M, K, N, kernel, splits):
    """Where reading every word costs less than waiting for the union, and
    where the row-load kernels are the faster ones."""
    p = plan(T, M, K, N, blocked=1)
    assert (p.status, p.kernel, p.splits) == (B.NMDLM_OK, kernel, splits)
    for option in ("bias", "cur", "theta_vec"):            # never with these
        assert plan(T, M, K, N, blocked=1, **{option: 1}).kernel != "lean"
    assert plan(T, M, K, N).kernel != "lean"               # nor without the copy


@pytest.mark.parametrize("T,M,K,N,kernel,rows", [
    (4, 13, 124, 10055, "words", 16),    # 632 workgroups, more than two per CU
    (8, 37, 106, 2841, "words", 16),
    (4, 13, 124, 8192, "lean", 16),      # 512
    (4, 13, 512, 10055, "lean", 32),     # a word for every wave: taller tiles
    (1, 325, 175, 3272, "words", 32),    # one step, 312 workgroups of 64 rows
    (1, 256, 175, 4096, "lean", 64),     # 256: one per CU, eight waves
    (1, 325, 175, 2600, "words", 16),    # 861 of 16
    (1, 325, 175, 4800, "lean", 64),     # 450
    (2, 163, 175, 3272, "lean", 64),     # two steps
])
def test_lean_with_few_words(T, M, K, N, kernel, rows):
    """K below 512 leaves lean waves idle: only where the grid fits at once."""
    p = plan(T, M, K, N, blocked=1)
    assert (p.status, p.kernel, p.rows) == (B.NMDLM_OK, kernel, rows)


@pytest.mark.parametrize("T,M,K,N,rows", [
    (4, 39, 14677, 5973, 32),    # 282 workgroups of 64 rows: two rounds, the third row block half empty
    (1, 134, 14024, 11963, 32),  # 561: three
    (8, 17, 7600, 5700, 32),     # 270
    (8, 17, 7400, 5700, 64),     # two workgroups a CU
    (7, 25, 15560, 10656, 64),   # 501: two rounds nearly full
    (4, 64, 14336, 4096, 64),    # 256: one
    (4, 64, 14336, 4160, 32),    # 260
])
def test_lean_rounds(T, M, K, N, rows):
    """64-row tiles, one workgroup on a CU, only where their rounds are full."""
    p = plan(T, M, K, N, blocked=1)
    assert (p.status, p.kernel, p.rows) == (B.NMDLM_OK, "lean", rows)


@pytest.mark.parametrize("T,M,K,N,kernel", [
    (4, 5200, 3000, 64, "lean"),      # 163 workgroups of one column tile
    (8, 1283, 3450, 273, "lean"),     # 162, five column tiles in two groups
    (8, 1283, 3450, 512, "tall"),     # 162 full ones
    (4, 5200, 1000, 64, "lean"),
    (4, 5200, 1000, 128, "tall"),     # 326 tiles
    (4, 5200, 500, 64, "tall"),
])
def test_tall_with_few_columns(T, M, K, N, kernel):
    p = plan(T, M, K, N, blocked=1)
    assert (p.status, p.kernel) == (B.NMDLM_OK, kernel)


@pytest.mark.parametrize("T,M,K,N,kernel,waves", [
    (5, 658, 4257, 8506, "words", 4),    # 7315 workgroups: four fit a CU, two of the lean ones
    (7, 612, 4414, 6434, "words", 4),
    (5, 104, 4257, 8506, "lean", 8),     # 1197
    (6, 196, 4443, 10994, "lean", 8),    # 70 words: three
    (7, 206, 4096, 12000, "lean", 8),    # 64 words
    (7, 36, 3975, 25067, "lean", 8),     # 63: two lean workgroups a CU, of eight waves
    (7, 36, 3960, 25067, "lean", 4),     # 62: three of four
])
def test_lean_residency(T, M, K, N, kernel, waves):
    p = plan(T, M, K, N, blocked=1)
    assert (p.status, p.kernel, p.rows, p.waves) == (B.NMDLM_OK, kernel, 64, waves)


def test_attention_route():
    """One kernel or two, and the parts of a timestep."""
    # one timestep: four parts of any context, while they run at once
    assert attn_route(1, 25, 7, 16, 128) == (1, 4, False)
    assert attn_route(1, 32, 700, 8, 128, step=1) == (1, 4, False)
    assert attn_route(1, 600, 0, 16, 64) == (1, 1, False)
    assert attn_route(2, 31, 480, 8, 128) == (1, 4, False)
    # many timesteps: a long walk of few workgroups is shared by eight waves
    assert attn_route(8, 31, 640, 8, 128) == (1, 1, True)
    assert attn_route(8, 100, 560, 16, 128) == (1, 1, False)     # 896 workgroups of k_attn
    # a step does not pay the host's pace for the second launch
    for T, M, C, H, dh in ((4, 7, 350, 8, 128), (5, 7, 150, 4, 128), (8, 7, 100, 4, 128), (8, 7, 350, 8, 64)):
        assert attn_route(T, M, C, H, dh) == (1, 1, False)
        assert attn_route(T, M, C, H, dh, step=1) == (1, 1, True)
        assert attn_route(T, M, C, H, dh, step=1, fused=1) == (1, 1, False)
    assert attn_route(4, 16, 512, 16, 64, step=1) == (1, 1, False)
    assert attn_route(4, 32, 1024, 16, 128, step=1) == (1, 2, True)
    assert attn_route(8, 16, 300, 16, 64, n_seq=4, step=1) == (1, 1, False)   # 512 workgroups of k_attn
