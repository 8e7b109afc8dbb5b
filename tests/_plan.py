"""The library's choice of a product's kernel (a host-side query: no GPU)."""
import ctypes as C
from types import SimpleNamespace

from paper_2607_24841_amd import binding as B

CUR, IF, QNL_IF, HEAD, BITWISE, MODIF = range(6)
KERNELS = ("list", "fused", "words", "wide", "dma", "lean", "tall")


class _Query(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("mode", "T", "M", "K", "N", "blocked", "bias", "cur", "theta_vec",
                                         "ternary", "theta", "transposed", "pos0", "seq_len")]
    _fields_ += [("flags", C.c_uint32)]


class _Answer(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("status", "kernel", "rows", "tokens", "row_blocks", "splits",
                                         "waves")]


def plan(T, M, K, N, mode=IF, theta=256, **options):
    """Kernel, rows and tokens of a row block, row blocks, K splits and waves of
    the product of these sizes; options as the fields of the query."""
    a = _Answer()
    B.load().nmdlm_internal_plan(C.byref(_Query(mode=mode, T=T, M=M, K=K, N=N, theta=theta, **options)),
                                 C.byref(a))
    return SimpleNamespace(status=a.status, kernel=KERNELS[a.kernel], rows=a.rows, tokens=a.tokens,
                           row_blocks=a.row_blocks, splits=a.splits, waves=a.waves)


def step_plans(T, M, d, F, pos0=0, n_seq=1, V=0):
    """The products of one layer of a block step over blocked copies (qkv, o,
    up, dn), and of the head where V > 0."""
    R = n_seq * M
    seq = M if n_seq > 1 else 0
    p = dict(qkv=plan(T, R, d, 3 * d, blocked=1, transposed=1, pos0=pos0, seq_len=seq),
             o=plan(T, R, d, d, blocked=1), up=plan(T, R, d, F, mode=QNL_IF, blocked=1),
             dn=plan(T, R, F, d, blocked=1))
    if V:
        p["head"] = plan(T, R, d, V, mode=HEAD, blocked=1)
    return p


def token_runs(pos0, seq_len, tokens, M, y):
    """Runs of row block y (of `tokens` of the M tokens) in a channel-major
    segment: (sequence, first position, tokens, stored in bytes)."""
    out = (C.c_int32 * (4 * tokens))()
    n = B.load().nmdlm_internal_token_runs(pos0, seq_len, tokens, M, y, out)
    return [tuple(out[4 * i:4 * i + 4]) for i in range(n)]


def attn_route(T, M, C_, H, dh, n_seq=1, fused=0, step=0):
    """(16-query groups of a wave, waves per timestep, attention and IF in two kernels)."""
    out = (C.c_int32 * 3)()
    B.load().nmdlm_internal_attn_route(T, M, C_, H, dh, n_seq, fused, step, out)
    return out[0], out[1], bool(out[2])
