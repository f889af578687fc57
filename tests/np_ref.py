"""Independent numpy helpers used only to pin the oracle (never as expected
values for the GPU path: those come from oracle/ alone).  They restate the
packed layout with array operations instead of the oracle's scalar loops, so a
wrong index or nibble order in the oracle shows up as a disagreement."""
import numpy as np


def unpack_codes(qweight: np.ndarray) -> np.ndarray:
    """u8 [N, K/2] -> signed codes int32 [N, K] (layout: byte g*16+j holds
    element 32g+j in its low nibble and element 32g+16+j in its high nibble)."""
    N, half = qweight.shape
    G = half // 16
    b = qweight.reshape(N, G, 16).astype(np.int32)
    lo = (b & 15) - 8
    hi = (b >> 4) - 8
    return np.concatenate([lo, hi], axis=2).reshape(N, G * 32)


def half_bits_to_f64(bits: np.ndarray) -> np.ndarray:
    return bits.astype(np.uint16).view(np.float16).astype(np.float64)


def bf16_bits_to_f64(bits: np.ndarray) -> np.ndarray:
    u = bits.astype(np.uint16).astype(np.uint32) << 16
    return u.view(np.float32).astype(np.float64)


def dequant(qweight: np.ndarray, scales: np.ndarray) -> np.ndarray:
    codes = unpack_codes(qweight).astype(np.float64)
    s = half_bits_to_f64(scales)
    return codes * np.repeat(s, 32, axis=1)


def rel_l2(a: np.ndarray, b: np.ndarray) -> float:
    a = np.asarray(a, np.float64).ravel()
    b = np.asarray(b, np.float64).ravel()
    d = np.linalg.norm(a - b)
    n = np.linalg.norm(b)
    return float(d / n) if n > 0 else float(d)


def sums_in_order(acc, sw, chains, xs=None, by_group=False):
    """float32 [M, N]: sum_g sw[n, g] * (xs[m, g]) * acc[m, n, g] in the order of the multi-token
    kernels, every step one fused multiply-add rounded to float32.  chains = 64: chain v takes groups
    v, v + 64, ..., and the chains are added in pairs, those 32 apart first; else chain v takes the
    columns (four groups) v, v + chains, ..., and the chains are added in order.  A scale per group
    (by_group) multiplies the weights' scale; one per token multiplies a chain's sum (columns) or the
    result.  (The steps are taken in 64-bit significands: rounding twice instead of once shows at
    one step in some 2^39.)"""
    M, N, G = acc.shape
    sw = np.asarray(sw, np.float32)
    xs = np.ones((M, G) if by_group else M, np.float32) if xs is None else np.asarray(xs, np.float32)
    f = np.zeros((chains, M, N), np.float32)
    for g in range(G):
        v = g % chains if chains == 64 else (g // 4) % chains
        s = np.broadcast_to(sw[None, :, g], (M, N))
        if by_group:
            s = s * xs[:, None, g]
        f[v] = (s.astype(np.longdouble) * acc[:, :, g] + f[v]).astype(np.float32)
    if chains == 64:
        while f.shape[0] > 1:
            h = f.shape[0] // 2
            f = f[:h] + f[h:]
        return f[0] if by_group else f[0] * xs[:, None]
    y = np.zeros((M, N), np.float32)
    for v in range(chains):
        y = y + (f[v] if by_group else f[v] * xs[:, None])
    return y


def sums_in_steps(acc, sw, xs=None):
    """float32 [M, N]: the same sum in the order of the persistent grid with shared activations: the
    eight groups of a step one after the other, the steps' sums eight at a time, then those."""
    M, N, G = acc.shape
    sw = np.asarray(sw, np.float32)
    zero = lambda: np.zeros((M, N), np.float32)
    total, f = zero(), zero()
    for c in range(G // 8):
        part = zero()
        for g in range(8 * c, 8 * c + 8):
            part = (sw[None, :, g].astype(np.longdouble) * acc[:, :, g] + part).astype(np.float32)
        f = f + part
        if c % 8 == 7:
            total, f = total + f, zero()
    total = total + f
    return total if xs is None else total * np.asarray(xs, np.float32)[:, None]
