"""CPU check of the attention normalisation's quotient: floor(256 num / den)
for 0 <= num <= den < 255 * 65536 taken as a float product with a lowered
reciprocal (correctly rounded, or one unit in the last place off either way, as
the hardware reciprocal may be) and one remainder correction equals the exact
integer quotient."""
import numpy as np


def test_lowered_estimate_is_exact():
    """The four-wide quotient: n * k with k = rcp(den) * 256 (1 - 2^-20),
    truncated, plus one when the fused remainder 256 n - q den reaches den."""
    rng = np.random.default_rng(13)
    dmax = 255 * 65535
    den = np.concatenate([np.arange(1, 4097), rng.integers(1, dmax + 1, 400000), np.full(4096, dmax),
                          255 * rng.integers(1, 65536, 100000), 2 ** rng.integers(0, 24, 4096)])
    num = np.minimum(np.floor(rng.random(den.size) * (den + 1)).astype(np.int64), den)
    num[:2048], num[2048:8192] = 0, den[2048:8192]
    k = rng.integers(0, 257, den.size)
    num[8192:200000] = ((k * den) // 256)[8192:200000]        # at and just below an integer quotient
    num[200000:300000] = np.maximum((k * den) // 256 - 1, 0)[200000:300000]
    exact = (256 * num) // den
    fn, fd = num.astype(np.float32), den.astype(np.float32)
    for shift in (0, 1, -1):
        r = (np.float32(1.0) / fd).astype(np.float32)
        if shift:
            r = np.nextafter(r, np.float32(np.inf if shift > 0 else 0)).astype(np.float32)
        scale = (r * np.float32(256.0 - 2.0 ** -12)).astype(np.float32)
        q = np.trunc((fn * scale).astype(np.float32))
        rem = 256.0 * num.astype(np.float64) - q.astype(np.float64) * den   # exact below 2^53
        got = q.astype(np.int64) + (rem.astype(np.float32) >= fd)
        assert np.array_equal(got, exact)
