"""Timed cases of the block-denoising library: what a program of this
framework calls, from the smallest product to a prefill, through the public
binding.  Inputs are drawn on the GPU from the seed; `exact` evaluates the
same inputs in float64 (every product sum is an integer below 2^53, so it is
exact) without the library.

Kinds of case
  qbsm     one spiking product, row-major weights or with the blocked copy
  attn     one spike-attention call followed by its IF neuron
  step     a block step (or, with C = 0 and no head, a context prefill)
           through some layers, for one or several sequences
  ternary  ternary coding of integer activations and the product on the planes
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2607_24841_amd import binding as B

DEV = "cuda"


# ----------------------------------------------------------------------------
# cases
# ----------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: one spiking linear layer, currents and spikes out
        dict(name="linear_512", kind="qbsm", T=4, M=8, K=512, N=512, rho=0.15, blocked=False,
             bias=True, cur=True, spk=True),
        # one token through an FFN up product at a sparse input (decode, row skipping)
        dict(name="ffn_up_b1", kind="qbsm", T=4, M=1, K=4096, N=14336, rho=0.05, blocked=True,
             bias=False, cur=False, spk=True),
        # a 64-token block through an FFN down product at a dense input
        dict(name="ffn_dn_b64", kind="qbsm", T=4, M=64, K=14336, N=4096, rho=0.30, blocked=True,
             bias=False, cur=False, spk=True),
        # sizes that fill no tile, three timesteps, row-major weights only
        dict(name="ragged_rows", kind="qbsm", T=3, M=37, K=1000, N=1500, rho=0.10, blocked=False,
             bias=True, cur=True, spk=True),
        # attention of an odd-sized block over an odd-sized context
        dict(name="attn_ragged", kind="attn", T=4, M=45, C=333, H=8, dh=64, cur=True),
        # attention of a whole prompt over itself (the prefill of the 24-layer model)
        dict(name="attn_prompt", kind="attn", T=4, M=2048, C=0, H=16, dh=128, cur=False),
        # one layer, 16 masked tokens over 512 context tokens (one-block step)
        dict(name="block_step", kind="step", layers=1, T=4, M=16, C=512, d=1024, H=16, F=4096, V=0,
             n_seq=1, tokens=False),
        # the same layer over 128 sequences at once (serving)
        dict(name="block_step_n128", kind="step", layers=1, T=4, M=16, C=512, d=1024, H=16, F=4096,
             V=0, n_seq=128, tokens=False),
        # prompt prefill, 2048 ids through two layers of the 24-layer model
        dict(name="prefill_2048", kind="step", layers=2, T=4, M=2048, C=0, d=2048, H=16, F=8192,
             V=0, n_seq=1, tokens=True),
        # the 12-layer denoising step with head, confidence and unmasking
        dict(name="mdlm12_step", kind="step", layers=12, T=4, M=32, C=1024, d=2048, H=16, F=8192,
             V=32000, n_seq=1, tokens=True),
        # a decoder step of the encoder-decoder shape: T = 8, a block of 4 tokens
        dict(name="e2d2_step", kind="step", layers=4, T=8, M=4, C=64, d=512, H=8, F=1536, V=32000,
             n_seq=1, tokens=True),
        # a converted layer: ternary coding of four tokens and the FFN up product
        dict(name="ternary_up", kind="ternary", T=8, M=4, K=4096, N=14336, levels=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the same ranges, at most the prefill's cost."""
    kind = rng.choice(["qbsm", "qbsm", "attn", "attn", "step", "step", "prefill", "ternary"])
    if kind == "qbsm":
        K = _log(rng, 64, 14336)
        N = _log(rng, 64, min(14336, (60 << 20) // K))
        return dict(kind="qbsm", T=rng.choice([1, 2, 3, 4, 4, 8]), M=_log(rng, 1, 96), K=K, N=N,
                    rho=round(math.exp(rng.uniform(math.log(0.02), math.log(0.3))), 3),
                    blocked=rng.random() < 0.6, bias=rng.random() < 0.5, cur=rng.random() < 0.5,
                    spk=True)
    if kind == "attn":
        T, dh = rng.choice([1, 2, 3, 4, 4, 8]), rng.choice([64, 128])
        H = rng.choice([4, 8, 12, 16])
        M = _log(rng, 1, 2048)
        C = rng.randrange(0, 1500)
        if T * M * (C + M) * H * dh > 4 * 2048 * 2048 * 16 * 128:
            C = 0
            M = min(M, 1024)
        return dict(kind="attn", T=T, M=M, C=C, H=H, dh=dh, cur=rng.random() < 0.5)
    if kind == "step":
        d = rng.choice([256, 512, 1024, 2048])
        T = rng.choice([1, 2, 4, 4, 8])
        n = rng.choice([1, 1, 1, 3, 8, 24, 64])
        M = _log(rng, 1, 48)
        if n > 1:
            M = max(16 // T, M // (16 // T) * (16 // T))
            d = min(d, 1024)
        V = rng.choice([0, 0, 5008, 32000]) if n * M <= 256 else 0
        return dict(kind="step", layers=rng.randrange(1, 4), T=T, M=M, C=_log(rng, 1, 1100), d=d,
                    H=d // rng.choice([64, 128]), F=16 * _log(rng, 16, 4 * d // 16), V=V, n_seq=n,
                    tokens=V > 0 or rng.random() < 0.5)
    if kind == "prefill":
        d = rng.choice([512, 1024, 2048])
        return dict(kind="step", layers=1, T=rng.choice([2, 4, 4, 8]), M=_log(rng, 64, 1600), C=0,
                    d=d, H=d // rng.choice([64, 128]), F=16 * _log(rng, d // 16, 4 * d // 16), V=0,
                    n_seq=1, tokens=rng.random() < 0.5)
    K = _log(rng, 256, 6000)
    return dict(kind="ternary", T=rng.choice([2, 4, 6, 8]), M=_log(rng, 1, 16), K=K,
                N=_log(rng, 64, 14336), levels=rng.randrange(1, 5))


# ----------------------------------------------------------------------------
# inputs, from the seed alone
# ----------------------------------------------------------------------------
def _gen(seed, *path):
    s = 1469598103934665603
    for v in (seed, *path):
        s = ((s ^ (int(v) + 1)) * 1099511628211) % (1 << 63)
    return torch.Generator(device=DEV).manual_seed(s)


def _i8(gen, *shape):
    return torch.randint(-127, 128, shape, dtype=torch.int8, device=DEV, generator=gen)


def _scaled_beta(rng, K, b, mean):
    """Per-channel spike rates ~ Beta(0.5, b), scaled to the given mean."""
    r = rng.beta(0.5, b, size=K)
    lo, hi = 0.0, 1.0
    while np.clip(hi * r, 0, 1).mean() < mean and hi < 1e9:
        hi *= 2
    for _ in range(60):
        mid = (lo + hi) / 2
        lo, hi = (mid, hi) if np.clip(mid * r, 0, 1).mean() < mean else (lo, mid)
    return np.clip(hi * r, 0, 1)


def _pack(bits):
    """Boolean [..., K] -> int64 words [..., ceil(K/64)], bit j of word w = channel 64 w + j."""
    K = bits.shape[-1]
    pad = -K % 64
    if pad:
        bits = torch.nn.functional.pad(bits, (0, pad))
    w = torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], dtype=torch.uint8, device=bits.device)
    by = (bits.reshape(-1, 8).to(torch.uint8) * w).sum(-1, dtype=torch.uint8)
    return by.view(torch.int64).reshape(*bits.shape[:-1], (K + pad) // 64)


def _unpack(words, K):
    by = words.reshape(-1).view(torch.uint8).reshape(*words.shape[:-1], -1, 1)
    sh = torch.arange(8, dtype=torch.uint8, device=words.device)
    return ((by >> sh) & 1).bool().reshape(*words.shape[:-1], -1)[..., :K]


def _table_u8(gen):
    return torch.randint(1, 256, (256,), device=DEV, generator=gen).sort().values.to(torch.uint8)


def _table_s8(gen):
    v = torch.randint(-128, 128, (256,), device=DEV, generator=gen).sort().values
    return torch.roll(v, 128).to(torch.int8).view(torch.uint8)  # indexed by the signed byte


def _qbsm_inputs(c, seed):
    rates = _scaled_beta(np.random.default_rng([seed, 1]), c["K"], 8.0, c["rho"])
    rates = torch.from_numpy(rates.astype(np.float32)).to(DEV)
    S = torch.rand(c["T"], c["M"], c["K"], device=DEV, generator=_gen(seed, 2)) < rates
    ldw = -(-c["N"] // 16) * 16
    W = _i8(_gen(seed, 3), c["K"], ldw)
    bias = torch.randint(-64, 65, (c["N"],), dtype=torch.int32, device=DEV, generator=_gen(seed, 4))
    return S, W, ldw, bias if c["bias"] else None, 256


def _attn_inputs(c, seed):
    d, cap = c["H"] * c["dh"], -(-(c["C"] + c["M"]) // 64) * 64
    q = torch.rand(c["T"], c["M"], d, device=DEV, generator=_gen(seed, 1)) < 0.4
    k = torch.rand(c["T"], cap, d, device=DEV, generator=_gen(seed, 2)) < 0.4
    v = torch.rand(c["T"], cap, d, device=DEV, generator=_gen(seed, 3)) < 0.4
    return q, k, v, cap, _table_u8(_gen(seed, 4)), 200


def _layer_inputs(c, seed, l):
    d, F = c["d"], c["F"]
    th = np.random.default_rng([seed, 5, l]).integers(128, 513, size=7)
    return SimpleNamespace(
        d=d, F=F, H=c["H"], dh=d // c["H"], W_qkv=_i8(_gen(seed, 10, l), d, 3 * d),
        W_o=_i8(_gen(seed, 11, l), d, d), W_up=_i8(_gen(seed, 12, l), d, F),
        W_dn=_i8(_gen(seed, 13, l), F, d), lut_att=_table_u8(_gen(seed, 14, l)),
        lut_act=_table_s8(_gen(seed, 15, l)), s_up=max(0, int(math.floor(math.log2(d))) - 6),
        theta={n: int(v) for n, v in zip(("q", "k", "v", "a", "o", "up", "dn"), th)})


def _caches(c, seed, l, cap):
    """Keys and values of the context: words [n_seq][T][cap][d/64] and, word-major,
    [n_seq][T][cap/64][d].  Rows past the context are empty."""
    n, T, d, C = c["n_seq"], c["T"], c["d"], c["C"]
    k = torch.zeros(n, T, cap, d // 64, dtype=torch.int64, device=DEV)
    vt = torch.zeros(n, T, cap // 64, d, dtype=torch.int64, device=DEV)
    for s in range(n if C else 0):
        b = torch.rand(2, T, C, d, device=DEV, generator=_gen(seed, 20, l, s)) < 0.4
        k[s, :, :C] = _pack(b[0])
        v = torch.zeros(T, cap, d, dtype=torch.bool, device=DEV)
        v[:, :C] = b[1]
        vt[s] = _pack(v.transpose(1, 2).contiguous()).transpose(1, 2)
    return k, vt


def _step_inputs(c, seed):
    n, T, M, d = c["n_seq"], c["T"], c["M"], c["d"]
    x = SimpleNamespace(cap=-(-(c["C"] + M) // 64) * 64, X=None, emb=None, pos_ch=None, tokens=None)
    if c["tokens"]:
        V = c["V"] or 32000
        rates = np.random.default_rng([seed, 1]).beta(0.5, 6.0, size=d).astype(np.float32)
        rates = torch.from_numpy(rates).to(DEV)
        g = _gen(seed, 2)
        x.emb = torch.cat([_pack(torch.rand(min(4000, V + 1 - v), T, d, device=DEV, generator=g) < rates)
                           for v in range(0, V + 1, 4000)])
        x.pos_ch = torch.randint(0, d, (c["C"] + M, T), dtype=torch.int32, device=DEV,
                                 generator=_gen(seed, 3))
        x.tokens = torch.randint(0, V, (n * M,), dtype=torch.int32, device=DEV, generator=_gen(seed, 4))
        # a step with the head starts from a block whose last tokens are masked
        x.masked = (torch.arange(n * M, device=DEV) % M >= (M // 4 if c["V"] else M)).to(torch.uint8)
    else:
        x.X = torch.rand(T, n * M, d, device=DEV, generator=_gen(seed, 6)) < 0.10
    if c["V"]:
        x.W_head = _i8(_gen(seed, 7), d, c["V"])
        x.scale = (0.5 + torch.rand(c["V"], device=DEV, generator=_gen(seed, 8))) * 2.0 ** -10
    return x


def _ternary_inputs(c, seed):
    """Integer activations: a few large channels, many small ones."""
    rng = np.random.default_rng([seed, 1])
    a = rng.laplace(0.0, 1.0, size=(c["M"], c["K"])) * rng.beta(0.5, 6.0, size=c["K"]) * 1000.0
    a = torch.from_numpy(np.rint(a).astype(np.int32)).to(DEV)
    return a, _i8(_gen(seed, 2), c["K"], -(-c["N"] // 16) * 16)


# ----------------------------------------------------------------------------
# the calls
# ----------------------------------------------------------------------------
def prepare(case, seed):
    c = case
    s = SimpleNamespace(c=c)
    if c["kind"] == "qbsm":
        S, s.W, s.ldw, s.bias, s.theta = _qbsm_inputs(c, seed)
        s.s_in = _pack(S)
        s.Wb = B.blocked_weights(s.W, c["K"], c["N"], s.ldw) if c["blocked"] else None
        s.cur = torch.empty(c["T"], c["M"], c["N"], dtype=torch.int32, device=DEV) if c["cur"] else None
        s.spk = torch.empty(c["T"], c["M"], -(-c["N"] // 64), dtype=torch.int64, device=DEV)
        s.stats = torch.zeros(4, dtype=torch.int64, device=DEV)
        s.ws = B.workspace(B.nmdlm_qbsm_workspace_size(c["T"], c["M"], c["K"], c["N"]))
    elif c["kind"] == "attn":
        q, k, v, s.cap, s.lut, s.theta = _attn_inputs(c, seed)
        s.q, s.k = _pack(q), _pack(k)
        s.vt = _pack(v.transpose(1, 2).contiguous()).transpose(1, 2).contiguous()
        d = c["H"] * c["dh"]
        s.a = torch.empty(c["T"], c["M"], d, dtype=torch.int32, device=DEV) if c["cur"] else None
        s.spk = torch.empty(c["T"], c["M"], d // 64, dtype=torch.int64, device=DEV)
        s.ws = B.workspace(B.nmdlm_bbm_attn_workspace_size(c["T"], c["M"], c["H"], c["dh"]))
    elif c["kind"] == "step":
        _prepare_step(s, c, seed)
    else:
        s.a, s.W = _ternary_inputs(c, seed)
        kw = -(-c["K"] // 64)
        s.pos = torch.empty(c["T"], c["M"], kw, dtype=torch.int64, device=DEV)
        s.neg = torch.empty_like(s.pos)
        s.sum = torch.empty(c["M"], dtype=torch.int64, device=DEV)
        s.acc = torch.empty(c["M"], c["N"], dtype=torch.int32, device=DEV)
        s.ws = B.workspace(B.nmdlm_qbsm_workspace_size(c["T"], c["M"], c["K"], c["N"]))
    return s


def _prepare_step(s, c, seed):
    x = _step_inputs(c, seed)
    n, T, M, d, head = c["n_seq"], c["T"], c["M"], c["d"], c["V"] > 0

    def host(L):
        return SimpleNamespace(**{k: v.cpu().numpy() if isinstance(v, torch.Tensor) else v
                                  for k, v in vars(L).items()})

    s.dm = B.DeviceModel(
        [host(_layer_inputs(c, seed, l)) for l in range(c["layers"])], T, x.cap, d, c["H"], c["F"],
        V=c["V"] or 32000, emb=None if x.emb is None else x.emb.cpu().numpy(),
        pos_ch=None if x.pos_ch is None else x.pos_ch.cpu().numpy(),
        W_head=x.W_head.cpu().numpy() if head else None,
        scale=x.scale.cpu().numpy() if head else None, max_seq=n, blocked=True)
    for l, L in enumerate(s.dm.layers):
        k, vt = _caches(c, seed, l, x.cap)
        L.k_seq.copy_(k)
        L.vt_seq.copy_(vt)
    flags = 0 if head else B.NMDLM_NO_HEAD
    s.ws = B.workspace(B.nmdlm_block_step_workspace_size(s.dm, n * M, flags))
    s.y = torch.empty(T, n * M, d // 64, dtype=torch.int64, device=DEV)
    s.x = None if x.X is None else _pack(x.X)
    s.tokens0, s.masked0 = x.tokens, getattr(x, "masked", None)
    s.tokens = None if x.tokens is None else x.tokens.clone()
    s.masked = None if x.tokens is None else x.masked.clone()
    k_unmask = max(1, M // 4)
    s.head = {}
    if head:
        s.head = dict(logits=torch.empty(n * M, c["V"], dtype=torch.float32, device=DEV),
                      pred=torch.empty(n * M, dtype=torch.int32, device=DEV),
                      conf=torch.empty(n * M, dtype=torch.float64, device=DEV),
                      unmasked_pos=torch.empty(n, k_unmask, dtype=torch.int32, device=DEV))
    s.io = B.step_io(M, c["C"], pos0=c["C"], flags=flags, x_in=s.x, tokens=s.tokens,
                     masked=s.masked, k_unmask=k_unmask if head else 0, y_out=s.y, n_seq=n, **s.head)


def run(s):
    c = s.c
    if c["kind"] == "qbsm":
        args = dict(bias=s.bias, cur_out=s.cur, theta=s.theta, s_out=s.spk, stats=s.stats, ws=s.ws)
        if s.Wb is not None:
            B.nmdlm_qbsm_blocked(s.s_in, c["T"], c["M"], c["K"], s.W, s.Wb, c["N"], s.ldw, **args)
        else:
            B.nmdlm_qbsm(s.s_in, c["T"], c["M"], c["K"], s.W, c["N"], s.ldw, **args)
        return [s.cur, s.spk, s.stats]
    if c["kind"] == "attn":
        B.nmdlm_bbm_attn(s.q, s.k, s.vt, s.cap, c["T"], c["M"], c["C"], c["H"], c["dh"], s.lut,
                         a_out=s.a, theta_a=s.theta, s_out=s.spk, ws=s.ws)
        return [s.a, s.spk]
    if c["kind"] == "step":
        if s.head:  # a block starts from its tokens and its masks
            s.tokens.copy_(s.tokens0)
            s.masked.copy_(s.masked0)
        B.nmdlm_block_step(s.dm, s.io, s.ws)
        out = dict(s.head, y=s.y, k=[L.k_seq for L in s.dm.layers], v=[L.vt_seq for L in s.dm.layers])
        if s.head:
            out.update(tokens=s.tokens, masked=s.masked)
        return out
    B.nmdlm_ternary_encode(s.a, c["M"], c["K"], c["levels"], c["T"], s.pos, s.neg, s.sum)
    B.nmdlm_qbsm_ternary(s.pos, s.neg, c["T"], c["M"], c["K"], s.W, c["N"], s.W.shape[1], s.acc,
                         ws=s.ws)
    return [s.pos, s.neg, s.sum, s.acc]


def _union_share(rates, draws):
    return float(np.mean(1.0 - (1.0 - rates) ** draws))


def work(case):
    """Weights of the rows that spike somewhere in the block (as expected from
    the inputs' rates; every row inside a step), each input and output once;
    two operations per spike row, active weight row and column."""
    c = case
    T, M = c["T"], c["M"]
    if c["kind"] == "qbsm":
        rows = c["K"] * _union_share(_scaled_beta(np.random.default_rng(0), c["K"], 8.0, c["rho"]), T * M)
        out = T * M * (4 * c["N"] * c["cur"] + c["N"] / 8)
        return dict(bytes=rows * c["N"] + T * M * c["K"] / 8 + out, flops=2 * T * M * rows * c["N"])
    if c["kind"] == "attn":
        d, J = c["H"] * c["dh"], c["C"] + M
        return dict(bytes=T * (2 * M + 2 * J) * d / 8 + 4 * T * M * d * c["cur"],
                    flops=2 * 2 * T * M * J * d)
    if c["kind"] == "step":
        n, d, F, J = c["n_seq"], c["d"], c["F"], c["C"] + M
        R = T * n * M
        w = 4 * d * d + 2 * d * F
        by = c["layers"] * (w + n * T * 2 * J * d / 8) + 2 * R * d / 8
        fl = c["layers"] * (2 * R * w + 4 * R * J * d)
        if c["V"]:
            by += d * c["V"] + n * M * c["V"] * 4
            fl += 2 * R * d * c["V"]
        return dict(bytes=by, flops=fl)
    r = c["K"] * 0.7  # channels that code to a nonzero value in some token
    return dict(bytes=4 * M * c["K"] + 2 * T * M * c["K"] / 8 + r * c["N"] + 4 * M * c["N"],
                flops=2 * T * M * r * c["N"])


def tolerance(case):
    """Spikes, currents and caches are integers: the same for every correct
    implementation.  Logits are one float32 product per entry, the confidence
    a float64 sum of their exponentials."""
    if case["kind"] == "step" and case["V"]:
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    return "exact"


# ----------------------------------------------------------------------------
# the same in 64 bits
# ----------------------------------------------------------------------------
def _if64(cur, theta, resid=None):
    V = torch.zeros_like(cur[0])
    out = []
    for t in range(cur.shape[0]):
        V = V + cur[t] + (0 if resid is None else theta * resid[t].double())
        s = V >= theta
        V = V - theta * s
        out.append(s)
    return torch.stack(out)


def _attn64(q, k, v, H, lut):
    """floor(256 sum_j p V / sum_j p) per head, p = lut[popcount(Q and K)]."""
    T, M, d = q.shape
    dh = d // H
    a = torch.zeros(T, M, d, dtype=torch.float64, device=DEV)
    for t in range(T):
        for h in range(H):
            c = slice(h * dh, (h + 1) * dh)
            p = lut.double()[(q[t, :, c].double() @ k[t, :, c].double().T).long()]
            num, den = (p @ v[t, :, c].double()).long(), p.sum(1, keepdim=True).long()
            a[t, :, c] = torch.where(den > 0, (256 * num) // den.clamp(min=1), 0).double()
    return a


def exact(case, seed):
    c = case
    T, M = c["T"], c["M"]
    if c["kind"] == "qbsm":
        S, W, _, bias, theta = _qbsm_inputs(c, seed)
        cur = S.double() @ W[:, :c["N"]].double()
        if bias is not None:
            cur = cur + bias
        act = int(S.any(0).any(0).sum())
        st = torch.tensor([c["K"], act, c["N"], act * c["N"]], dtype=torch.int64)
        return [cur.int() if c["cur"] else None, _pack(_if64(cur, theta)), st]
    if c["kind"] == "attn":
        q, k, v, _, lut, theta = _attn_inputs(c, seed)
        J = c["C"] + M
        a = _attn64(q, k[:, :J], v[:, :J], c["H"], lut)
        return [a.int() if c["cur"] else None, _pack(_if64(a, theta))]
    if c["kind"] == "step":
        return _exact_step(c, seed)
    a, W = _ternary_inputs(c, seed)
    al = a.long()
    S = al.abs().sum(1)
    DK = c["K"] * c["levels"]
    mag = (2 * al.abs() * DK + S[:, None]) // (2 * S[:, None]).clamp(min=1)
    mag = torch.where(S[:, None] > 0, mag, 0).clamp(max=(1 << T) - 1)
    bits = torch.stack([((mag >> t) & 1).bool() for t in range(T)])
    acc = (al.sign() * mag).double() @ W[:, :c["N"]].double()
    return [_pack(bits & (a > 0)), _pack(bits & (a < 0)), S, acc.int()]


def _exact_step(c, seed):
    x = _step_inputs(c, seed)
    n, T, M, d, C, H = c["n_seq"], c["T"], c["M"], c["d"], c["C"], c["H"]
    X = x.X
    if X is None:
        ids = torch.where(x.masked.bool(), c["V"], x.tokens).long()
        X = _unpack(x.emb[ids].transpose(0, 1), d).clone()
        pos = x.pos_ch[C:C + M].repeat(n, 1).T.long()  # [T][n M]
        X.scatter_(2, pos[..., None], True)
    ks, vs = [], []
    for l in range(c["layers"]):
        L = _layer_inputs(c, seed, l)
        th = L.theta
        qkv = X.double() @ L.W_qkv.double()
        q, k, v = (_if64(qkv[..., i * d:(i + 1) * d], th[p]) for i, p in enumerate("qkv"))
        kc, vt = _caches(c, seed, l, x.cap)
        A = torch.empty(T, n * M, d, dtype=torch.float64, device=DEV)
        for s in range(n):
            r = slice(s * M, (s + 1) * M)
            kc[s, :, C:C + M] = _pack(k[:, r])
            vb = _unpack(vt[s].transpose(1, 2).contiguous(), x.cap).transpose(1, 2).contiguous()
            vb[:, C:C + M] = v[:, r]
            vt[s] = _pack(vb.transpose(1, 2).contiguous()).transpose(1, 2)
            kb = _unpack(kc[s], d)
            A[:, r] = _attn64(q[:, r], kb[:, :C + M], vb[:, :C + M], H, L.lut_att)
        A = _if64(A, th["a"])
        X1 = _if64(A.double() @ L.W_o.double(), th["o"], X)
        u = torch.floor((X1.double() @ L.W_up.double()) / 2.0 ** L.s_up).clamp(-128, 127).long()
        h = _if64(L.lut_act.view(torch.int8).double()[u & 255], th["up"])
        X = _if64(h.double() @ L.W_dn.double(), th["dn"], X1)
        ks.append(kc)
        vs.append(vt)
    out = dict(y=_pack(X), k=ks, v=vs)
    if c["V"]:
        lg = (X.sum(0, dtype=torch.float64) @ x.W_head.double()) * x.scale.double()
        # which tokens are revealed follows from the logits' float32 rounding at ties
        out.update(logits=lg, conf=torch.softmax(lg, 1).max(1).values, pred=None, unmasked_pos=None,
                   tokens=None, masked=None)
    return out
