"""Oracle of the initial vacuum fluctuations (TEST INFRASTRUCTURE ONLY: only
tests/, the smoke entry and the benchmark's CPU baseline use it).

Sainio, arXiv:0911.5692, Sec. II.B: the homogeneous field values are inputs
and the random fluctuations are generated by the program through an FFT, as
in DEFROST; the fields are then in program units (f = A a^r phi) and the
velocities are the rescaled physical ones, u = (A/B) a^(r-s) dphi/dt, to
which the Friedmann initialisation adds r (a'/a) f.

Readings taken where the paper only cites the method:
  * spectrum of each field fluctuation P(k) = eps^2 / (2 omega_k) and of each
    velocity fluctuation eps^2 omega_k / 2, omega_k = sqrt(k^2 + m_i^2), the
    four arrays statistically independent; k = 2 pi n / L, the k = 0 mode and
    every |n| above the cutoff (default N/4) removed;
  * lattice normalisation: a white-noise array w of unit variance is filtered
    as f = IFFT( FFT(w) * sqrt(N^3 P(k) / L^3) ), so that
    <f^2> = sum_k P(k) / L^3;
  * the white noise is drawn with the counter-based generator Philox4x32-10
    (Salmon, Moraes, Dror, Shaw, "Parallel random numbers: as easy as 1, 2,
    3", SC'11): for site i (linear index, x fastest) of array j
    (f1, f2, u1, u2 = 0..3) the counter is (i mod 2^32, i div 2^32, j, 0) and
    the key (seed mod 2^32, seed div 2^32); its four output words
    x0..x3 give two uniforms in (0, 1] with 53 random bits, exact in FP64,
        U1 = (x0 * 2^21 + floor(x1 / 2^11) + 1) / 2^53,
        U2 = (x2 * 2^21 + floor(x3 / 2^11) + 1) / 2^53,
    and the Box-Muller normal sqrt(-2 ln U1) cos(2 pi U2).
Everything is FP64; numpy's FFT is a library step.
"""
from __future__ import annotations

import numpy as np

_M0, _M1 = np.uint64(0xD2511F53), np.uint64(0xCD9E8D57)
_W0, _W1 = 0x9E3779B9, 0xBB67AE85
_MASK = np.uint64(0xFFFFFFFF)


def philox4x32_10(c0, c1, c2, c3, k0: int, k1: int):
    """Philox4x32 with 10 rounds (SC'11 definition): each round multiplies
    words 0 and 2 by the two round constants, takes the 64-bit products'
    high halves xor the other two words and the round key, and the round key
    is bumped by the Weyl constants between rounds.  Vectorised over the
    counter words (uint32 arrays or scalars); returns four uint32 arrays."""
    c = [np.asarray(v, dtype=np.uint64) & _MASK for v in (c0, c1, c2, c3)]
    ka, kb = int(k0) & 0xFFFFFFFF, int(k1) & 0xFFFFFFFF
    for r in range(10):
        p0 = _M0 * c[0]
        p1 = _M1 * c[2]
        hi0, lo0 = p0 >> np.uint64(32), p0 & _MASK
        hi1, lo1 = p1 >> np.uint64(32), p1 & _MASK
        c = [hi1 ^ c[1] ^ np.uint64(ka), lo1, hi0 ^ c[3] ^ np.uint64(kb), lo0]
        ka, kb = (ka + _W0) & 0xFFFFFFFF, (kb + _W1) & 0xFFFFFFFF
    return [v.astype(np.uint32) for v in c]


def uniform53(hi, lo):
    """(hi * 2^21 + lo // 2^11 + 1) / 2^53 in (0, 1], exact in FP64."""
    m = (np.asarray(hi, dtype=np.uint64) << np.uint64(21)) | (np.asarray(lo, dtype=np.uint64) >> np.uint64(11))
    return (m + np.uint64(1)).astype(np.float64) * 2.0 ** -53


def white_noise(N: int, seed: int, j: int, sites=None) -> np.ndarray:
    """Unit normal noise of array j at every site (shape (N, N, N)) or at the
    given linear site indices."""
    i = np.arange(N ** 3, dtype=np.uint64) if sites is None else np.asarray(sites, dtype=np.uint64)
    x0, x1, x2, x3 = philox4x32_10(i & _MASK, i >> np.uint64(32), np.full(i.shape, j, np.uint64),
                                   np.zeros(i.shape, np.uint64), seed & 0xFFFFFFFF, seed >> 32)
    u1, u2 = uniform53(x0, x1), uniform53(x2, x3)
    g = np.sqrt(-2.0 * np.log(u1)) * np.cos(2.0 * np.pi * u2)
    return g.reshape(N, N, N) if sites is None else g


def mode_norm(N: int) -> np.ndarray:
    """|n| of every rfftn mode, n the FFT-signed integer wavevector.  Whole
    numbers: fftfreq(N) * N misses some by a rounding (9, 13 and 18 at N = 125),
    which would decide whether a mode at the cutoff is kept."""
    n0 = np.rint(np.fft.fftfreq(N) * N)
    n2 = np.rint(np.fft.rfftfreq(N) * N)
    return np.sqrt(n0[:, None, None] ** 2 + n0[None, :, None] ** 2 + n2[None, None, :] ** 2)


def spectrum(N: int, L: float, m2: float, eps2: float, kind: str, cutoff: float | None = None):
    """P(k) on the rfftn grid (zero at k = 0 and above the cutoff)."""
    cutoff = N / 4 if cutoff is None or cutoff == 0 else cutoff
    nn = mode_norm(N)
    omega = np.sqrt((2.0 * np.pi * nn / L) ** 2 + m2)
    P = eps2 / (2.0 * omega) if kind == "field" else eps2 * omega / 2.0
    P[(nn == 0) | (nn > cutoff)] = 0.0
    return P


def fluctuation(N: int, L: float, m2: float, eps2: float, kind: str, seed: int, j: int,
                cutoff: float | None = None) -> np.ndarray:
    """Gaussian random field of array j with the vacuum spectrum of its kind."""
    W = np.fft.rfftn(white_noise(N, seed, j))
    W *= np.sqrt(N ** 3 * spectrum(N, L, m2, eps2, kind, cutoff) / L ** 3)
    return np.fft.irfftn(W, s=(N, N, N), axes=(0, 1, 2))


def vacuum_state(N: int, L: float, f0, u0, m2, eps2: float, seed: int, cutoff: float | None = None) -> dict:
    """f_i = f0_i + field fluctuation (array i), u_i = u0_i + velocity
    fluctuation (array 2 + i), i = 1, 2; program units, FP64."""
    out = {}
    for i in range(2):
        out[f"f{i + 1}"] = f0[i] + fluctuation(N, L, m2[i], eps2, "field", seed, i, cutoff)
        out[f"u{i + 1}"] = u0[i] + fluctuation(N, L, m2[i], eps2, "velocity", seed, 2 + i, cutoff)
    return out
