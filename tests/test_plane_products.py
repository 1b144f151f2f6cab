"""The factor's large products on two fp16 planes an operand, emulated on the CPU: what they leave
of a factor's accuracy, and that a lost low plane is far above the tolerance of the GPU tests."""
import numpy as np
import pytest

# Relative Frobenius error against 64 bits of U and of its block between the two parts of a node.
# The emulation below leaves 3.6e-7 to 5.0e-7 (as fp32 products do: the sums in fp32 decide it);
# four times that. A lost low plane of one operand leaves 2e-4.
PLANE_TOL = 2e-6

D, HALF = 1536, 768


def _planes(a, lost):
    """High and low fp16 parts of a, rows scaled by powers of two to a largest value in [2^14, 2^15)."""
    a = a.astype(np.float32)
    top = np.abs(a).max(axis=1, keepdims=True)
    unit = np.exp2(np.floor(np.log2(np.where(top > 0, top, 1.0))) - 14).astype(np.float32)
    x = a / unit
    hi = x.astype(np.float16).astype(np.float32)
    lo = (x - hi).astype(np.float16).astype(np.float32)
    return hi, np.zeros_like(lo) if lost else lo, unit


def _product(p, q):
    """P Q^T by three fp32 products of planes."""
    (ph, pl, pu), (qh, ql, qu) = p, q
    return (pl @ qh.T + ph @ ql.T + ph @ qh.T) * pu * qu.T


def _inverse_factor(m):
    n = len(m)
    if n <= 96:
        return np.linalg.inv(np.linalg.cholesky(m))
    h = n // 2
    x11 = _inverse_factor(m[:h, :h])
    l21 = m[h:, :h] @ x11.T
    x22 = _inverse_factor(m[h:, h:] - l21 @ l21.T)
    x = np.zeros((n, n))
    x[:h, :h], x[h:, h:], x[h:, :h] = x11, x22, -x22 @ (l21 @ x11)
    return x


def _off_block(M, lost=None):
    """The block X21 of L^-1 (M = L L^T), one node of two halves; leaves in float64, rounded."""
    m32 = M.astype(np.float32)
    x11 = _inverse_factor(m32[:HALF, :HALF].astype(np.float64)).astype(np.float32)
    pl = lambda a, name: _planes(np.ascontiguousarray(a), name == lost)
    l21 = _product(pl(m32[HALF:, :HALF], "M21"), pl(x11, "X11"))
    p = pl(l21, "L21")
    m22 = m32[HALF:, HALF:] - _product(p, p)
    t = _product(p, pl(x11.T, "X11^T"))
    x22 = _inverse_factor(m22.astype(np.float64)).astype(np.float32)
    return -_product(pl(x22, "X22"), pl(t.T, "T"))


def _matrix(sigma):
    rng = np.random.default_rng(1)
    if sigma is None:
        X = rng.standard_normal((2 * D, D))
        return (X.T @ X / (2 * D)).astype(np.float32).astype(np.float64)
    A = np.triu(rng.standard_normal((D, D)) * sigma, 1)
    return (np.eye(D) + A + A.T).astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("sigma", [None, 2e-3, 1e-4, 1e-6])
def test_plane_products_error(sigma):
    M = _matrix(sigma)
    ref = _inverse_factor(M)[HALF:, :HALF]
    err = lambda lost: np.linalg.norm(_off_block(M, lost) - ref) / np.linalg.norm(ref)
    assert err(None) < PLANE_TOL / 3
    # (with a coupling of 1e-4 or less the low planes of X are below the sums' rounding)
    for lost in ("M21", "L21", "T") + (("X11", "X11^T", "X22") if sigma in (None, 2e-3) else ()):
        assert err(lost) > 20 * PLANE_TOL, lost
