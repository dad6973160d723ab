"""What fp32 contractions are held to: the relative error of a plain chain of fp32 multiply-adds over the same operands."""
import numpy as np


def rel(a, b):
    return np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b)


def chain(a, b):
    """a . b with one fp32 rounding per multiply-add, in order."""
    a, b = a.astype(np.float64), b.astype(np.float64)
    acc = np.zeros((a.shape[0], b.shape[1]))
    for k in range(a.shape[1]):
        acc = (acc + a[:, k:k + 1] * b[k:k + 1]).astype(np.float32).astype(np.float64)
    return acc


def reference(a, b):
    """(a . b in 64 bits, the chain's error against it)"""
    ref = a.astype(np.float64) @ b.astype(np.float64)
    return ref, rel(chain(a, b), ref)


# ---- the operations as products of matrices (k4 s2 p1; images [n, side, side, channels], filters [16, cb, cs])

def columns_down(big):
    """Rows: output pixels; columns: (tap, channel)."""
    n, side, _, cb = big.shape
    hs = side // 2
    p = np.zeros((n, side + 2, side + 2, cb), big.dtype)
    p[:, 1:-1, 1:-1] = big
    return np.concatenate([p[:, ky:ky + side:2, kx:kx + side:2].reshape(n * hs * hs, cb) for ky in range(4) for kx in range(4)], 1)


def columns_up(small):
    """Rows: pixels of the larger map; columns: (tap, channel), zero where a tap does not meet the pixel."""
    n, hs, _, cs = small.shape
    p = np.zeros((n, 2 * hs + 4, 2 * hs + 4, cs), small.dtype)
    p[:, 2:2 + 2 * hs:2, 2:2 + 2 * hs:2] = small              # position 2 y + 2
    return np.concatenate([p[:, 3 - ky:3 - ky + 2 * hs, 3 - kx:3 - kx + 2 * hs].reshape(-1, cs) for ky in range(4) for kx in range(4)], 1)


# ---- the arithmetic of fp32 storage: values as three bf16 parts, six products, sums of sixteen products rounded to fp32

def _bf16(x):
    u = np.ascontiguousarray(x, np.float32).view(np.uint32).astype(np.uint64)
    return (((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16).astype(np.uint32).view(np.float32)


def _parts(x, scale):
    x = np.float32(x) * np.float32(scale)
    h = _bf16(x)
    m = _bf16(x - h)
    return h, m, _bf16(x - h - m)


SMALL = ((2, 0), (0, 2), (1, 1), (1, 0), (0, 1))               # (part of a, part of b), 0 the largest


def split_product(a, b, scale=2.0 ** 24, small=SMALL):
    A, B = _parts(a, scale), _parts(b, scale)
    acc = np.zeros((a.shape[0], b.shape[1]), np.float32)
    low = acc.copy()
    for k in range(0, a.shape[1], 16):
        def product(i, j):
            return A[i][:, k:k + 16].astype(np.float64) @ B[j][k:k + 16].astype(np.float64)
        for i, j in small:
            low = (low + product(i, j)).astype(np.float32)
        acc = (acc + product(0, 0)).astype(np.float32)
    return (acc + low) * np.float32(1.0 / scale) * np.float32(1.0 / scale)
