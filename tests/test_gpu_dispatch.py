"""Each branch of the size-dependent dispatches at its edges, against the float64 oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import synth
from gpu_util import DEV, note, rel_frob, rot_device, rot_oracle, to_np
from paper_2607_07964_amd import kronq as K
from test_plane_products import PLANE_TOL

pytestmark = pytest.mark.gpu


# ---------------------------------------------------------------- fp32 covariance tile sizes
# 16-, 32- and 64-edge tiles (the largest that gives every CU a workgroup), token counts below,
# at and past the 16-wave shares, ragged channel counts, row strides past d
@pytest.mark.parametrize("cross", [False, True])
@pytest.mark.parametrize("n,d", [(1, 1), (3, 17), (130, 256), (2049, 257), (515, 530), (77, 1030),
                                 (1000, 1100), (129, 1601)])
def test_cov_fp32_tiles(n, d, cross):
    rng = np.random.default_rng(n * 7 + d)
    a = rng.standard_normal((n, d + 3)).astype(np.float32)
    b = rng.standard_normal((n, d + 3)).astype(np.float32) if cross else a
    h0 = rng.standard_normal((d, d)).astype(np.float32)
    A, B = torch.from_numpy(a).to(DEV)[:, :d], torch.from_numpy(b).to(DEV)[:, :d]
    note(f"cov fp32 n={n} d={d} cross={cross}")
    for beta in (0.0, 0.5):
        H = torch.from_numpy(h0).to(DEV) if beta else torch.full((d, d), float("nan"), device=DEV)
        ws = torch.empty(256, dtype=torch.uint8, device=DEV)
        if cross:
            K.kronq_accumulate_cross(A, B, H, 2.0, beta, ws)
        else:
            K.kronq_accumulate_cov(A, H, 2.0, beta, ws)
        torch.cuda.synchronize()
        ref = 2.0 * (a[:, :d].astype(np.float64).T @ b[:, :d].astype(np.float64)) + beta * h0
        # n-term fp32 sums of the products: n 2^-24 of the sum of the terms' sizes at most
        size = 2.0 * (np.abs(a[:, :d]).astype(np.float64).T @ np.abs(b[:, :d])) + np.abs(beta * h0)
        assert np.all(np.abs(to_np(H) - ref) <= (n + 4) * 2.0 ** -24 * size)
        if not cross and beta == 0.0:
            assert np.array_equal(to_np(H), to_np(H).T)


# ------------------------------------------------------- packed-code GEMV: widths and batches
# one group of columns (seven waves without work), group counts that leave waves short of a tile,
# the LDS limit (4 x 8192), several row blocks per workgroup, ragged last row block
@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("d_out,d_in,group,batch", [
    (1, 128, 128, 1), (17, 128, 128, 3), (33, 1152, 1152, 2), (40, 4224, 384, 3),
    (48, 8192, 256, 4), (8200, 256, 128, 4), (50, 8192, 128, 1), (20, 28672, 128, 1)])
def test_online_gemv_widths(d_out, d_in, group, batch, bits):
    rng = np.random.default_rng(d_out + d_in + bits)
    codes = rng.integers(0, 2 ** bits, size=(d_out, d_in)).astype(np.uint8)
    scales = (rng.random((d_out, d_in // group)) + 0.5).astype(np.float32)
    zeros = rng.integers(0, 2 ** bits, size=(d_out, d_in // group)).astype(np.float32)
    x = rng.standard_normal((batch, d_in)).astype(np.float32)
    x[:, ::97] *= 50.0  # outliers set their group's exponent
    note(f"gemv {d_out}x{d_in} group={group} batch={batch} bits={bits}")
    packed = K.kronq_pack_codes(torch.from_numpy(codes).to(DEV), bits)
    assert d_in * bits // 32 % 4 == 0  # whole 16-byte units, as the call asks
    y = K.kronq_online_matvec(packed, torch.from_numpy(scales).to(DEV),
                              torch.from_numpy(zeros).to(DEV), bits, group, d_in, None, None, None,
                              None, torch.from_numpy(x).to(DEV), flags=0)
    torch.cuda.synchronize()
    w = (codes.reshape(d_out, -1, group) - zeros[..., None].astype(np.float64)) * scales[..., None]
    w = w.reshape(d_out, d_in)
    ref = x.astype(np.float64) @ w.T
    # digits: 2^-30 of a group's largest x' per element; fp32 sums over d_in / 128 groups and two
    # roundings per term, of terms whose sizes add up to |x| (q + z) s
    size = np.abs(x.astype(np.float64)) @ ((codes.reshape(d_out, -1, group)
                                            + np.abs(zeros)[..., None] + 128.0 * (bits == 8))
                                           * scales[..., None]).reshape(d_out, d_in).T
    assert np.all(np.abs(to_np(y) - ref) <= (d_in // 128 + 8) * 2.0 ** -24 * size)


def test_online_gemv_nonfinite_input():
    """A NaN in one vector reaches all of its outputs and none of another vector's."""
    packed = torch.zeros(32, 256 * 4 // 32, dtype=torch.int32, device=DEV)
    sc, ze = torch.ones(32, 2, device=DEV), torch.ones(32, 2, device=DEV)
    x = torch.ones(2, 256, device=DEV)
    x[1, 7] = float("nan")
    note("gemv NaN")
    y = to_np(K.kronq_online_matvec(packed, sc, ze, 4, 128, 256, None, None, None, None, x,
                                    flags=0))
    assert np.all(y[0] == -256.0) and np.all(np.isnan(y[1]))


# ------------------------------------------------------------------ sweep: row groups and ties
def _solve(W, U, bits, group, P=None, err=False):
    d_out, d_in = W.shape
    Wd, Ud = (torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in (W, U))
    codes = torch.empty(d_out, d_in, dtype=torch.uint8, device=DEV)
    sc, ze = (torch.empty(d_out, d_in // group, device=DEV) for _ in range(2))
    E, Wh = torch.empty_like(Wd), torch.empty_like(Wd)
    if P is None:
        K.kronq_obs_quantize_layer(Wd, Ud, bits, codes, sc, ze, E if err else None, Wh, group)
    else:
        K.kronq_obs_quantize_layer_drift(Wd, Ud, torch.from_numpy(np.ascontiguousarray(P)).to(DEV), bits, codes, sc, ze,
                                         E if err else None, Wh, group)
    torch.cuda.synchronize()
    return {k: to_np(v) for k, v in dict(codes=codes, scales=sc, zeros=ze, W=Wd, w_hat=Wh,
                                         err=E).items()}


# one and two row groups per workgroup (beyond 64 and, with P, 32 rows per CU), a ragged last
# group of 32 rows, an idle second row group; lazy groups of 1 to 4 blocks, partly filled
@pytest.mark.parametrize("d_out,d_in,group,drift", [
    (1, 128, 128, False), (33, 640, 128, True), (31, 768, 384, False), (64, 1280, 1280, True),
    (70, 1280, 640, False), (16417, 256, 128, False), (8225, 256, 128, True),
    (20000, 384, 384, False)])
def test_sweep_row_groups(d_out, d_in, group, drift):
    rng = np.random.default_rng(d_out + d_in)
    X = rng.standard_normal((4 * d_in, d_in))
    U = O.inverse_cholesky_factor(O.damp(X.T @ X)).astype(np.float32)
    P = None
    if drift:
        P = (np.triu(rng.standard_normal((d_in, d_in)), 1) * 0.02).astype(np.float32)
    W = (rng.standard_normal((d_out, d_in)) * 0.02).astype(np.float32)
    note(f"sweep {d_out}x{d_in} group={group} drift={drift}")
    got = _solve(W, U, 4, group, P, err=True)
    ref = O.obs_blocked(W, U, 4, group, 128, P=P)
    # fp32 rounding moves near ties; all that follows in such a row moves with them
    same = np.all(got["codes"] == ref["codes"], axis=1)
    assert np.mean(got["codes"] == ref["codes"]) > 0.9999 and np.mean(same) > 0.99
    assert np.allclose(got["scales"][same], ref["scales"][same], rtol=1e-5)
    assert np.array_equal(got["zeros"][same], ref["zeros"][same])
    assert rel_frob(got["err"][same], ref["err"][same]) < 1e-4
    assert np.array_equal(got["W"], got["w_hat"])
    g = np.repeat(np.arange(d_in // group), group)
    deq = got["scales"][:, g] * (got["codes"].astype(np.float32) - got["zeros"][:, g])
    assert np.array_equal(got["w_hat"], deq)


def test_sweep_exact_ties():
    """Values on and one ulp beside the half-integers of a power-of-two and of another scale, with
    U = I (no compensation): the codes are those of the exact quotient, ties to even."""
    rng = np.random.default_rng(5)
    rows, bits = 96, 4
    scale = np.where(np.arange(rows) % 2 == 0, 0.25, rng.uniform(0.1, 0.3, rows)).astype(np.float32)
    n = rng.integers(0, 15, size=(rows, 128))
    W = ((n + 0.5).astype(np.float64) * scale[:, None]).astype(np.float32)
    kick = rng.integers(-1, 2, size=W.shape)
    W = np.where(kick > 0, np.nextafter(W, np.float32(9)), W)
    W = np.where(kick < 0, np.nextafter(W, np.float32(0)), W).astype(np.float32)
    W[:, 0], W[:, 1] = 0.0, (15.0 * scale.astype(np.float64)).astype(np.float32)
    note("sweep exact ties")
    got = _solve(W, np.eye(128, dtype=np.float32), bits, 128)
    ref = O.obs_blocked(W, np.eye(128), bits, 128, 128)
    assert np.array_equal(got["codes"], ref["codes"])


# trailing products: 64-, 128- and 256-edge tiles, halving over a number of lazy groups that is
# no power of two, one product per lazy group for a wide group that is none either; the oracle
# takes a sample of the rows (they are independent)
@pytest.mark.parametrize("d_out,d_in,group,drift", [
    (300, 1920, 640, False), (290, 2944, 128, True), (5001, 2688, 128, False),
    (24901, 1152, 128, False), (24901, 1152, 1152, True), (3000, 2048, 1024, False)])
def test_sweep_trailing_products(d_out, d_in, group, drift):
    rng = np.random.default_rng(d_out + d_in)
    X = rng.standard_normal((4 * d_in, d_in))
    U = O.inverse_cholesky_factor(O.damp(X.T @ X)).astype(np.float32)
    P = None
    if drift:
        P = (np.triu(rng.standard_normal((d_in, d_in)), 1) * 0.01).astype(np.float32)
    W = (rng.standard_normal((d_out, d_in), dtype=np.float32) * np.float32(0.02))
    note(f"sweep {d_out}x{d_in} group={group} drift={drift}")
    got = _solve(W, U, 4, group, P, err=True)
    rows = np.unique(np.concatenate([[0, d_out - 1], rng.choice(d_out, 200)]))
    ref = O.obs_blocked(W[rows], U, 4, group, 128, P=P)
    same = np.all(got["codes"][rows] == ref["codes"], axis=1)
    assert np.mean(got["codes"][rows] == ref["codes"]) > 0.999 and np.mean(same) > 0.9
    assert rel_frob(got["err"][rows][same], ref["err"][same]) < 1e-3


# ------------------------------------------------------------------ factor: products on planes
def _split_at(d):
    """Columns of the first part of an order-d node, which starts at the last column."""
    return -(-d // 128) // 2 * 128


def _factor(H, damp=0.01):
    d = H.shape[0]
    Hd = torch.from_numpy(np.ascontiguousarray(H, dtype=np.float32)).to(DEV)
    U = torch.full((d, d), float("nan"), device=DEV)
    info = K.kronq_cholesky_inv(Hd, U, damp)
    torch.cuda.synchronize()
    return to_np(U), int(info.item())


# the smallest large node (two halves of 768), ragged second halves, nested large nodes, orders
# that are no multiple of 4 (scalar copies), and a diagonal graded over twelve decades, which the
# normalisation takes out before the fp16 planes
@pytest.mark.parametrize("d,graded", [(1535, False), (1536, False), (1700, True), (2331, False),
                                      (3105, True)])
def test_factor_planes(d, graded):
    rng = np.random.default_rng(d)
    X = rng.standard_normal((2 * d, d))
    C = X.T @ X / (2 * d)
    s = 10.0 ** rng.uniform(-6, 6, d) if graded else np.ones(d)
    H = (C * s[:, None] * s[None, :]).astype(np.float32)
    note(f"factor d={d} graded={graded}")
    U, info = _factor(H, 0.0 if graded else 0.01)
    assert info == 0 and np.array_equal(U, np.triu(U))
    H64 = H.astype(np.float64) / s[:, None] / s[None, :]
    ref = O.inverse_cholesky_factor(H64 if graded else O.damp(H64))
    # (test_plane_products.py: what these products leave, and that a lost low plane is 40 times it)
    got = U * s[None, :]
    r = d - _split_at(d)
    assert rel_frob(got, ref) < PLANE_TOL
    assert rel_frob(got[:r, r:], ref[:r, r:]) < PLANE_TOL


# two parts that hardly depend on each other: the block of U between them is small beside the
# diagonal, and as accurate as the rest
@pytest.mark.parametrize("sigma", [2e-3, 1e-4, 1e-6])
def test_factor_planes_weak_coupling(sigma):
    d = 1536
    rng = np.random.default_rng(3)
    A = np.triu(rng.standard_normal((d, d)) * sigma, 1)
    H = (np.eye(d) + A + A.T).astype(np.float32)
    note(f"factor weak coupling {sigma}")
    U, info = _factor(H, 0.0)
    ref = O.inverse_cholesky_factor(H.astype(np.float64))
    r = d - _split_at(d)
    assert info == 0 and rel_frob(U, ref) < PLANE_TOL
    assert rel_frob(U[:r, r:], ref[:r, r:]) < PLANE_TOL


# Three channels [[1, 1, 1/2], [1, 1 + 2^-22, 1/2 + 2^-12], [1/2, 1/2 + 2^-12, 1/2 + 2^-22]] in an
# identity, damp 0: every step of the elimination is exact in fp32 (pivots 1, 2^-22, 2^-22) and the
# inverse factor has entries up to 2^21. In either half of the two parts, and in both.
@pytest.mark.parametrize("at", [(10, 200, 700), (800, 1000, 1500), (10, 900, 1400),
                                (10, 700, 1400)])
def test_factor_planes_wide_inverse(at):
    d = 1536
    trio = np.array([[1, 1, 0.5], [1, 1 + 2.0 ** -22, 0.5 + 2.0 ** -12],
                     [0.5, 0.5 + 2.0 ** -12, 0.5 + 2.0 ** -22]])
    idx = d - 1 - np.array(at)  # (the factorisation runs from the last column to the first)
    H = np.eye(d, dtype=np.float32)
    H[np.ix_(idx, idx)] = trio
    assert np.array_equal(H[np.ix_(idx, idx)].astype(np.float64), trio)
    L = np.linalg.cholesky(trio)
    X = np.zeros((3, 3))
    for j in range(3):  # L X = I by forward substitution
        for i in range(j, 3):
            X[i, j] = ((i == j) - L[i, :i] @ X[:i, j]) / L[i, i]
    ref = np.eye(d)
    ref[np.ix_(idx, idx)] = X
    note(f"factor wide inverse {at}")
    U, info = _factor(H, 0.0)
    assert info == 0 and np.abs(X).max() >= 2.0 ** 21
    np.testing.assert_allclose(U, ref, rtol=1e-6, atol=0)


def test_factor_planes_ragged_256_tiles():
    """An order whose large products all take 256-edge tiles, with ragged last rows (its parts are
    5760 and 5740): U H~ U^T is the identity."""
    d = 11500
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    X = torch.randn(2 * d, d, generator=g, device=DEV)
    H = X.T @ X / (2 * d)
    del X
    U = torch.full((d, d), float("nan"), device=DEV)
    note(f"factor 256 tiles d={d}")
    info = K.kronq_cholesky_inv(H, U, 0.01)  # (H becomes H~)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    U64 = U.double()
    R = U64 @ H.double() @ U64.T
    R.diagonal().sub_(1.0)
    # a relative error e of U leaves 2 e |U| |H~| |U| at most, a low plane lost 100 times it
    assert float(R.norm() / d ** 0.5) < 4 * PLANE_TOL and float(R.abs().max()) < 4 * PLANE_TOL
    assert not torch.tril(U, -1).any()


@pytest.mark.parametrize("d,bad", [(1536, 3), (1536, 1500), (2304, 900)])
def test_factor_planes_not_positive(d, bad):
    rng = np.random.default_rng(bad)
    X = rng.standard_normal((2 * d, d))
    H = X.T @ X / (2 * d)
    H[bad, bad] = -1.0
    note(f"factor d={d} bad={bad}")
    # the factorisation runs from the last column to the first: the first failure it meets
    assert _factor(H, 0.0)[1] == bad + 1


# ---------------------------------------------------------------- drift correction on fp16 planes
# orders on both sides of the planes' threshold, ragged tiles, padded rows, rows of D and U over
# many powers of two
@pytest.mark.parametrize("d,pad", [(1279, 1), (1280, 0), (1444, 0), (1539, 5)])
def test_gptaq_planes(d, pad):
    rng = np.random.default_rng(d)
    U = (np.triu(rng.standard_normal((d, d))) * 2.0 ** rng.integers(-12, 13, (d, 1))).astype(np.float32)
    D = (rng.standard_normal((d, d)) * 2.0 ** rng.integers(-12, 13, (d, 1))).astype(np.float32)
    D[d // 3] = 0.0
    dev = [torch.full((d, d + pad), float("nan"), device=DEV) for _ in range(3)]
    Dd, Ud, P = (t[:, :d] for t in dev)
    Dd.copy_(torch.from_numpy(D))
    Ud.copy_(torch.from_numpy(U))
    note(f"gptaq planes d={d} pad={pad}")
    K.kronq_gptaq_correction(Dd, Ud, P, 0.5)
    torch.cuda.synchronize()
    p = to_np(P)
    assert np.all(np.tril(p) == 0.0)
    D64, U64 = np.triu(D.astype(np.float64), 1), U.astype(np.float64)
    T = np.triu(D64 @ U64.T, 1)
    ref = 0.5 * T @ U64
    # two d-term fp32 sums of operands of 23 bits (2^-23 each) of the terms' sizes; an operand below
    # 2^-16 of its row's largest value (D and U with U's columns brought to one size, T, U's
    # columns) is good to 2^-39 of that (sizes to a power of two: a factor of two)
    top = lambda a, axis: np.abs(a).max(axis, keepdims=True)
    c = top(U64, 0)
    size = np.triu(np.abs(D64) @ np.abs(U64).T, 1)
    eT = (d + 12) * 2.0 ** -24 * size + d * 2.0 ** -37 * top(D64 * c, 1) * top(U64 / c, 1).T
    eP = (d + 12) * 2.0 ** -24 * size @ np.abs(U64) + d * 2.0 ** -38 * top(T, 1) * top(U64, 0)
    assert np.all(np.abs(p - ref) <= 0.5 * np.triu(np.triu(eT, 1) @ np.abs(U64) + eP, 1))
    if pad:
        assert torch.isnan(dev[2][:, d:]).all()


@pytest.mark.parametrize("d", [1279, 1280, 1539])
def test_gptaq_planes_graded_channels(d):
    """Channels of sizes over eight decades, as without the rescaling: D grows with both of its
    channels, U falls with its column's. P[p, n] is s_p / s_n times that of equal channels."""
    rng = np.random.default_rng(d)
    s = 10.0 ** rng.uniform(-4, 4, d)
    X = rng.standard_normal((2 * d, d))
    U = (O.inverse_cholesky_factor(O.damp(X.T @ X / (2 * d))) / s[None, :]).astype(np.float32)
    D = (rng.standard_normal((d, d)) * 0.1 * s[:, None] * s[None, :]).astype(np.float32)
    P = torch.empty(d, -(-d // 4) * 4, device=DEV)[:, :d]
    dev = [torch.zeros(d, -(-d // 4) * 4, device=DEV)[:, :d] for _ in range(2)]
    for t, a in zip(dev, (D, U)):
        t.copy_(torch.from_numpy(a))
    note(f"gptaq graded channels d={d}")
    K.kronq_gptaq_correction(dev[0], dev[1], P, 1.0)
    torch.cuda.synchronize()
    ref = np.triu(np.triu(D.astype(np.float64) @ U.astype(np.float64).T, 1) @ U, 1)
    w = s[None, :] / s[:, None]
    # (fp32 products leave 5e-7; the planes without factors per channel leave 1e-4)
    assert rel_frob(to_np(P) * w, ref * w) < PLANE_TOL


def test_gptaq_planes_ragged_256_tiles():
    """The 256-edge tiles of both products, with a ragged last tile; sampled rows in 64 bits."""
    d = 8004
    g = torch.Generator(device=DEV)
    g.manual_seed(2)
    U = torch.randn(d, d, generator=g, device=DEV).mul_(d ** -0.5).triu_()
    U.diagonal().add_(1.0)
    D = torch.randn(d, d, generator=g, device=DEV)
    P = torch.full((d, d), float("nan"), device=DEV)
    note(f"gptaq 256 tiles d={d}")
    K.kronq_gptaq_correction(D, U, P, 1.0)
    torch.cuda.synchronize()
    assert not torch.tril(P).any()
    rows = torch.tensor([0, 1, 255, 256, 4095, 5000, 7679, 7680, 7935, 7936, 8001, 8002], device=DEV)
    keep = torch.arange(d, device=DEV)[None, :] > rows[:, None]
    T = (D[rows].double() @ U.double().T) * keep
    ref = (T @ U.double()) * keep
    err = (P[rows].double() - ref).norm(dim=1) / ref.norm(dim=1)
    assert float(err.max()) < PLANE_TOL  # (a low plane lost: 2e-4)


# ---------------------------------------------------------------- rotations with a fused H_8
# both sides of the rule (2048 ... 8192 rows of 2048 or 4096), and its neighbours that keep two
# column passes (a row of 1024) or take one (1024 rows); W as bf16 and fp32, padded rows
@pytest.mark.parametrize("d_out,d_in,bf16", [(2048, 4096, True), (4096, 2048, False), (2048, 1024, False),
                                             (8192, 2048, True), (1024, 4096, True)])
def test_rotate_fused_rows(d_out, d_in, bf16):
    rng = np.random.default_rng(d_out + d_in)
    w = torch.from_numpy(rng.standard_normal((d_out, d_in)).astype(np.float32))
    w = w.to(torch.bfloat16) if bf16 else w
    hx, hg = (torch.from_numpy(rng.standard_normal((n, n)).astype(np.float32)) for n in (d_in, d_out))
    for h in (hx, hg):
        h += h.T.clone()
        h.diagonal().copy_(1.0 + torch.from_numpy(rng.random(h.shape[0]).astype(np.float32)))
    ri, ro = (synth.rotation_params(n, 5, s) for n, s in ((d_in, "in"), (d_out, "out")))
    rin, rout = rot_device(ri), rot_device(ro)
    wide = torch.full((d_out, d_in + 8), float("nan"), device=DEV)
    W, HX, HG = wide[:, :d_in], hx.to(DEV), hg.to(DEV)
    sx, sg = torch.empty(d_in, device=DEV), torch.empty(d_out, device=DEV)
    note(f"rotate fused rows {d_out}x{d_in} bf16={bf16}")
    K.kronq_rotate(w.to(DEV), W, HX, HG, rin.sign, rout.sign, rin.q28, rout.q28, sx, sg, K.BIIP)
    back = torch.empty(d_out, d_in, device=DEV)
    K.kronq_rotate(W, back, None, None, rin.sign, rout.sign, rin.q28, rout.q28, sx, sg,
                   K.BIIP | K.INVERSE)
    torch.cuda.synchronize()
    # a butterfly stage adds at most 2^-24 of the norm, the multipliers and norms a few more; a
    # sampled block's share of the error's norm is within 4 of its share of the norm
    tol = 4 * (np.log2(d_out) + np.log2(d_in) + 8) * 2.0 ** -24
    rows, cols = (np.sort(rng.choice(n, 24, replace=False)) for n in (d_out, d_in))
    sx64, sg64 = to_np(sx).astype(np.float64), to_np(sg).astype(np.float64)
    V = O.rht_rows(d_in, *rot_oracle(ri), cols)
    U = O.rht_rows(d_out, *rot_oracle(ro), rows)
    w64 = w.float().numpy().astype(np.float64)
    assert rel_frob(to_np(W)[np.ix_(rows, cols)], (U * sg64) @ w64 @ (V * sx64).T) < tol
    for got, h, t in ((HX, hx, V / sx64), (HG, hg, U / sg64)):
        idx = cols if got is HX else rows
        assert rel_frob(to_np(got)[np.ix_(idx, idx)], t @ h.numpy().astype(np.float64) @ t.T) < tol
    assert rel_frob(to_np(back), w64) < tol
    assert torch.isnan(wide[:, d_in:]).all()


# ------------------------------------------- rotations whose lane stages end before 512 elements
# rows of 28 * 128 and 28 * 256 (seven and eight stages in the lanes), one and several rows a
# workgroup, W as bf16 and fp32, both directions
@pytest.mark.parametrize("d_out,d_in,bf16", [(64, 3584, True), (2048, 3584, False), (256, 7168, True),
                                             (3584, 128, False)])
def test_rotate_short_lane_stages(d_out, d_in, bf16):
    rng = np.random.default_rng(d_out + d_in)
    w = torch.from_numpy(rng.standard_normal((d_out, d_in)).astype(np.float32))
    w = w.to(torch.bfloat16) if bf16 else w
    ri, ro = (synth.rotation_params(n, 5, s) for n, s in ((d_in, "in"), (d_out, "out")))
    rin, rout = rot_device(ri), rot_device(ro)
    X = rng.standard_normal((32, max(d_in, d_out)))
    hx, hg = ((X[:, :n].T @ X[:, :n] / 32 + np.eye(n)).astype(np.float32) for n in (d_in, d_out))
    W, HX, HG = torch.empty(d_out, d_in, device=DEV), *(torch.from_numpy(h).to(DEV) for h in (hx, hg))
    sx, sg = torch.empty(d_in, device=DEV), torch.empty(d_out, device=DEV)
    note(f"rotate short lane stages {d_out}x{d_in} bf16={bf16}")
    K.kronq_rotate(w.to(DEV), W, HX, HG, rin.sign, rout.sign, rin.q28, rout.q28, sx, sg, K.BIIP)
    back = torch.empty(d_out, d_in, device=DEV)
    K.kronq_rotate(W, back, None, None, rin.sign, rout.sign, rin.q28, rout.q28, sx, sg,
                   K.BIIP | K.INVERSE)
    torch.cuda.synchronize()
    # as above; the 28-point mix adds the rounding of 28-term sums
    tol = 4 * (np.log2(d_out) + np.log2(d_in) + 8 + 2 * np.sqrt(28)) * 2.0 ** -24
    rows, cols = (np.sort(rng.choice(n, 24, replace=False)) for n in (d_out, d_in))
    sx64, sg64 = to_np(sx).astype(np.float64), to_np(sg).astype(np.float64)
    V = O.rht_rows(d_in, *rot_oracle(ri), cols)
    U = O.rht_rows(d_out, *rot_oracle(ro), rows)
    w64 = w.float().numpy().astype(np.float64)
    assert rel_frob(to_np(W)[np.ix_(rows, cols)], (U * sg64) @ w64 @ (V * sx64).T) < tol
    for got, h, t, idx in ((HX, hx, V / sx64, cols), (HG, hg, U / sg64, rows)):
        assert rel_frob(to_np(got)[np.ix_(idx, idx)], t @ h.astype(np.float64) @ t.T) < tol
    assert rel_frob(to_np(back), w64) < tol


# Whole numbers without rescaling: every sum is exact in fp32, and so is the factor 1 / sqrt(d_out
# d_in) where it is a power of two, however the passes share it; the results have no error at all.
@pytest.mark.parametrize("d_out,d_in", [(4096, 4096), (2048, 2048), (8192, 2048), (1024, 4096)])
def test_rotate_exact_norm(d_out, d_in):
    rng = np.random.default_rng(d_out + d_in)
    w = rng.integers(-7, 9, size=(d_out, d_in)).astype(np.float32)
    ri, ro = (synth.rotation_params(n, 5, s) for n, s in ((d_in, "in"), (d_out, "out")))
    rin, rout = rot_device(ri), rot_device(ro)
    one_in, one_out = torch.ones(d_in, device=DEV), torch.ones(d_out, device=DEV)
    HX, W = torch.eye(d_in, device=DEV), torch.empty(d_out, d_in, device=DEV)
    note(f"rotate exact norm {d_out}x{d_in}")
    wd = torch.from_numpy(w).to(DEV)
    flags = K.ROT_IN | K.ROT_OUT
    K.kronq_rotate(wd, W, HX, None, rin.sign, rout.sign, rin.q28, rout.q28, one_in, one_out, flags)
    back = torch.empty_like(W)
    K.kronq_rotate(wd, back, None, None, rin.sign, rout.sign, rin.q28, rout.q28, one_in, one_out,
                   flags | K.INVERSE)
    torch.cuda.synchronize()
    rows, cols = (np.sort(rng.choice(n, 24, replace=False)) for n in (d_out, d_in))
    V, U = (np.rint(O.rht_matrix(n, *rot_oracle(r)) * np.sqrt(n)) for n, r in ((d_in, ri), (d_out, ro)))
    w64, norm = w.astype(np.float64), np.sqrt(d_out * d_in)
    assert np.array_equal(to_np(W)[np.ix_(rows, cols)], U[rows] @ w64 @ V[cols].T / norm)
    assert np.array_equal(to_np(back)[np.ix_(rows, cols)], U[:, rows].T @ w64 @ V[:, cols] / norm)
