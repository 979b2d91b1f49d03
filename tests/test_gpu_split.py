"""The split-precision fused pass against float64, where its tiling, packing
and scaling can go wrong: queries around the 16-, 64-, 128- and 256-row edges,
centres around the 128-row panel, features around the 32-feature step and the
points where the accumulated sign turns, label tiles of 16 full and one past,
rows of very different scale, and rows that are not 16-byte aligned."""

import numpy as np
import pytest

import oracle
from gpu_common import Gpu, TOL_STEP, bw32, kernel_id, rel

EPS = 2.0 ** -24


def _bound(X, Z, a, kernel, bw):
    """Elementwise bound of a float32 evaluation of K(Z, X) a: the squared
    distance |x|^2 + |z|^2 - 2 x.z is off by at most a few roundings of its
    terms (norms and dot product rounded, the dot product accumulated over
    d / 32 instructions of three products each, its scaled operands good to
    2^-22), the kernel value by that times its derivative (the Laplacian's
    at the smallest distance the error allows) and a few roundings of exp2 /
    sqrt, the sum over centres by its terms times the depth of a chain."""
    d = X.shape[1]
    xn, zn = (X.astype(np.float64) ** 2).sum(1), (Z.astype(np.float64) ** 2).sum(1)
    d2 = np.maximum(zn[:, None] + xn[None] - 2.0 * Z.astype(np.float64) @ X.T.astype(np.float64), 0)
    e2 = (6 + np.sqrt(d) / 4) * EPS * (zn[:, None] + xn[None])
    if kernel == "gaussian":
        K = np.exp(-d2 / (2 * bw * bw))
        dK = K * (e2 / (2 * bw * bw) + 8 * EPS * (1 + d2 / (2 * bw * bw)))
    else:
        r = np.sqrt(d2)
        K = np.exp(-r / bw)
        dr = np.minimum(np.sqrt(e2), e2 / np.maximum(r, 1e-300))
        dK = K * (np.expm1(dr / bw) + 8 * EPS * (1 + r / bw))
    chain = (8 + np.sqrt(X.shape[0])) * EPS
    return (dK + chain * K) @ np.abs(a.astype(np.float64)) + 1e-30


# Passes of at most 2^27 multiply-adds (queries counted in tiles of 64) take
# the float32 pass: n is large enough that these do not, and sits on, one
# past or one short of a 128-row panel.
CASES = [
    # kernel, n, d, l, n_z
    ("gaussian", 128 * 513, 32, 16, 64), ("laplacian", 128 * 250 + 1, 33, 17, 65),
    ("gaussian", 128 * 530 - 1, 32, 1, 1), ("laplacian", 128 * 45, 95, 15, 256),
    ("gaussian", 128 * 36 + 1, 97, 32, 257), ("gaussian", 128 * 65 + 1, 128, 33, 128),
    ("laplacian", 128 * 64 - 1, 129, 48, 129), ("gaussian", 128 * 52, 160, 160, 127),
    ("laplacian", 128 * 35 + 4, 161, 144, 130), ("gaussian", 128 * 16 + 2, 1030, 100, 63),
    ("gaussian", 300000, 7, 3, 65), ("laplacian", 128 * 9 - 2, 416, 80, 300),
    ("gaussian", 128 * 19 + 64, 224, 65, 250), ("laplacian", 128 * 2 + 1, 2500, 10, 320),
    ("gaussian", 100, 8200, 20, 200),
    # beyond 160 labels the kernel values are stored: label panels of 128
    # full, one tile past, one label past; several centre groups per split
    ("gaussian", 128 * 41 + 1, 100, 161, 250), ("laplacian", 128 * 60, 70, 256, 257),
    ("gaussian", 128 * 33 + 65, 135, 257, 300), ("gaussian", 128 * 8 - 1, 1040, 1100, 129),
    ("laplacian", 70000, 31, 500, 30),
]


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,n,d,l,n_z", CASES)
@pytest.mark.parametrize("law", ["normal", "positive", "scales"])
def test_predict_edges(kernel, n, d, l, n_z, law):
    assert -(-n_z // 64) * 64 * n * d > 2 ** 27
    rng = np.random.default_rng(n + d)
    X = rng.standard_normal((n, d)).astype(np.float32)
    Z = rng.standard_normal((n_z, d)).astype(np.float32)
    if law == "positive":
        X, Z = np.abs(X), np.abs(Z)
    if law == "scales":          # rows from 2^-30 to 2^10, zero rows among them
        X *= np.exp2(rng.integers(-30, 11, (n, 1))).astype(np.float32)
        Z *= np.exp2(rng.integers(-30, 11, (n_z, 1))).astype(np.float32)
        X[::17] = 0
        Z[::13] = 0
    Z[0] = X[n // 2]             # a repeated row
    a = (rng.standard_normal((n, l)) * np.exp2(rng.integers(-20, 3, (n, 1)))).astype(np.float32)
    bw = bw32(np.sqrt(d) * (0.8 if kernel == "gaussian" else 0.6))
    with Gpu(X, l, kernel, bw, min(n, 20), 2, np.arange(min(n, 20))) as g:
        g.set_alpha(a)
        P = g.predict(Z)
    P_o = oracle.predict(X.astype(np.float64), a.astype(np.float64), Z.astype(np.float64),
                         kernel_id(kernel), bw)
    b = _bound(X, Z, a, kernel, bw)
    worst = np.max(np.abs(P - P_o) / b)
    assert worst <= 1.0, worst


@pytest.mark.gpu
@pytest.mark.parametrize("m", [63, 64, 65, 128, 129, 255, 256, 257, 400])
@pytest.mark.parametrize("d,l", [(699, 12), (700, 30), (703, 200)])
def test_step_batch_edges(m, d, l):
    """Own centres (k = 1), kept subsample columns and the planes of alpha
    after each update, over two steps."""
    n, s, k, bw = 3001, 150, 12, bw32(1.3)
    rng = np.random.default_rng(m)
    X = (rng.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    Y = np.eye(l, dtype=np.float32)[rng.integers(0, l, n)]
    a0 = (rng.standard_normal((n, l)) / np.sqrt(n)).astype(np.float32)
    r = rng.choice(n, s, replace=False)
    st = oracle.setup(X, oracle.GAUSSIAN, bw, s, k, r)
    assert -(-m // 64) * 64 * n * d > 2 ** 27
    a_o = a0
    with Gpu(X, l, "gaussian", bw, s, k, r) as g:
        g.set_alpha(a0)
        for _ in range(2):
            t = rng.choice(n, m, replace=False)
            F = g.step(t, Y[t])
            a_n, F_o = oracle.step(st, a_o, t, Y[t])
            assert rel(F, F_o) < TOL_STEP
            a_o = a_n
        assert rel(g.alpha() - a0, a_o - a0) < TOL_STEP


@pytest.mark.gpu
@pytest.mark.parametrize("l", [3, 17, 160])
@pytest.mark.parametrize("n_z", [1, 16, 31, 32, 33, 63, 64, 65, 127, 128, 129])
def test_few_rows(l, n_z):
    """Tiles of 32, 64 and 128 rows whose waves share the queries and split
    the centres, and the reduction over many slices of few elements."""
    n, d, bw = 128 * 300 + 5, 64, bw32(7.0)
    rng = np.random.default_rng(n_z + l)
    X = rng.standard_normal((n, d)).astype(np.float32)
    Z = rng.standard_normal((n_z, d)).astype(np.float32)
    a = rng.standard_normal((n, l)).astype(np.float32)
    assert -(-n_z // 64) * 64 * n * d > 2 ** 27
    with Gpu(X, l, "gaussian", bw, 20, 2, np.arange(20)) as g:
        g.set_alpha(a)
        P = g.predict(Z)
    P_o = oracle.predict(X.astype(np.float64), a.astype(np.float64), Z.astype(np.float64),
                         oracle.GAUSSIAN, bw)
    assert np.max(np.abs(P - P_o) / _bound(X, Z, a, "gaussian", bw)) <= 1.0


@pytest.mark.gpu
@pytest.mark.parametrize("l", [9, 300])
@pytest.mark.parametrize("n_z", [3, 700])
def test_noalloc_in_chunks(l, n_z):
    """ep_predict_noalloc on the split pass, whose scratch holds the packed
    rows, the partial sums and (300 labels) the kernel values of a chunk."""
    import paper_1806_06144_amd as ep
    n, d, bw = 40001, 90, bw32(9.0)
    rng = np.random.default_rng(n_z + l)
    X = rng.standard_normal((n, d)).astype(np.float32)
    Z = rng.standard_normal((n_z, d)).astype(np.float32)
    a = rng.standard_normal((n, l)).astype(np.float32)
    assert -(-n_z // 64) * 64 * n * d > 2 ** 27
    with Gpu(X, l, "gaussian", bw, 20, 2, np.arange(20)) as g:
        g.set_alpha(a)
        out = g.torch.full((n_z, l), float("nan"), dtype=g.torch.float32, device=g.dev)
        ep.ep_predict_noalloc(g.ctx, g.t(Z), n_z, out)
        ep.ep_sync(g.ctx)
        P = out.cpu().numpy()
    P_o = oracle.predict(X.astype(np.float64), a.astype(np.float64), Z.astype(np.float64),
                         oracle.GAUSSIAN, bw)
    assert np.max(np.abs(P - P_o) / _bound(X, Z, a, "gaussian", bw)) <= 1.0


@pytest.mark.gpu
@pytest.mark.parametrize("s,m,k,l", [(63, 64, 1, 3), (64, 65, 20, 4), (65, 129, 21, 70),
                                     (500, 256, 63, 5), (1000, 300, 64, 33), (257, 4100, 65, 9)])
def test_correction_chunks(s, m, k, l):
    """Steps 4-5 in chunks of one accumulation block (s m <= 2^21), ragged in
    every dimension: alpha after one step."""
    n, d, bw = 4300, 20, bw32(1.1)
    rng = np.random.default_rng(s + m)
    X = (rng.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    Y = np.eye(l, dtype=np.float32)[rng.integers(0, l, n)]
    a0 = (rng.standard_normal((n, l)) / np.sqrt(n)).astype(np.float32)
    r = rng.choice(n, s, replace=False)
    t = rng.choice(n, m, replace=False)
    st = oracle.setup(X, oracle.GAUSSIAN, bw, s, min(k, s - 1), r)
    a_o, _ = oracle.step(st, a0, t, Y[t])
    with Gpu(X, l, "gaussian", bw, s, min(k, s - 1), r) as g:
        g.set_alpha(a0)
        g.step(t, Y[t])
        assert rel(g.alpha() - a0, a_o - a0) < TOL_STEP


def _rows(law, d, n, rng):
    if law == "two":             # 0 or a value midway between two fp16 numbers
        return (rng.random((n, d)) < 0.5) * np.float32(1.0 + 2.0 ** -11 + 2.0 ** -13)
    x = rng.standard_normal((n, d)).astype(np.float32)
    if law.startswith("column"):
        value, at = law.split()[1:]
        x[:, int(float(at) * (d - 1))] = np.float32(value)
    if law == "spread":          # features of very different size
        x *= np.exp2(-np.random.default_rng(d).integers(0, 21, d)).astype(np.float32)
    if law == "sparse":          # few features, so no sum evens the rounding out
        x *= rng.random((n, d)) < 12.0 / d
    return x.astype(np.float32)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [16, 64, 784])
@pytest.mark.parametrize("law", ["normal", "two", "spread", "sparse", "column 64.0312 0", "column 64.0312 1",
                                 "column 33.015 0.5", "column 65.03 0", "near"])
def test_distances_are_as_good_as_float32(law, d):
    """Squared distances, read off the kernel values of single centres, of
    rows that share large values or lie close together: their error against
    float64 is no larger than that of a float32 chain over the features, in
    the worse of two orders (a large value met first costs every later addition
    a rounding at its size), neither its root mean square nor its mean, which
    would move all kernel values alike. Allowed beside it: what packing a row
    to 2^-23 adds (computed from the packed values) and, as an accumulator of
    the 16-bit matrix cores is truncated where the chain is rounded, a tenth."""
    n, nz, l = int(2 ** 27 / (256 * d) * 1.3) + 77, 256, 32
    rng = np.random.default_rng(d)
    X = _rows("normal" if law == "near" else law, d, n, rng)
    Z = _rows("normal" if law == "near" else law, d, nz, rng)
    pair = np.ones((nz, l), dtype=bool)
    if law == "near":
        Z = (X[np.arange(nz) % l] + 2.0 ** -9 * rng.standard_normal((nz, d))).astype(np.float32)
        pair = np.arange(nz)[:, None] % l == np.arange(l)[None]
    x, z = X[:l], Z
    d2 = np.stack([((z.astype(np.float64) - r) ** 2).sum(1) for r in x.astype(np.float64)], 1)
    xn, zn = (x.astype(np.float64) ** 2).sum(1), (z.astype(np.float64) ** 2).sum(1)
    unit = EPS * (zn[:, None] + xn[None])
    pair &= unit > 0

    def chain(order):            # norms rounded from float64, one rounding a product
        dot = np.zeros((nz, l), dtype=np.float32)
        for j in order:
            dot = (dot + z[:, j, None].astype(np.float64) * x[None, :, j]).astype(np.float32)
        return (zn.astype(np.float32)[:, None] + xn.astype(np.float32)[None]) - np.float32(2) * dot

    # distance of the packed rows
    def packed(r):
        e = np.exp2(14 - np.floor(np.log2(np.abs(r).max(1, keepdims=True) + 1e-30))).astype(np.float32)
        h = (r * e).astype(np.float16).astype(np.float32)
        return (h.astype(np.float64) + (r * e - h).astype(np.float16)) / e

    p2 = np.stack([((packed(z) - r) ** 2).sum(1) for r in packed(x)], 1)
    bw = bw32(np.sqrt(d2[pair].mean() / 8))
    a = np.zeros((n, l), dtype=np.float32)
    a[np.arange(l), np.arange(l)] = 1.0
    assert -(-nz // 64) * 64 * n * d > 2 ** 27
    with Gpu(X, l, "gaussian", bw, 20, 2, np.arange(100, 120)) as g:
        g.set_alpha(a)
        K = g.predict(Z).astype(np.float64)
    scale = np.float64(np.float32(np.log2(np.e) / (2 * bw * bw)))
    ok = pair & (K > 0)
    assert ok.sum() > 0.9 * pair.sum()
    err = ((-np.log2(K[ok]) / scale) - d2[ok]) / unit[ok]
    ref = [(chain(order)[ok] - d2[ok]) / unit[ok] for order in (range(d), range(d - 1, -1, -1))]
    # what reading a distance off its kernel value adds: the rounding of exp2's
    # argument (uniform, 0.3 of its unit) and of exp2 (0.6)
    read = np.sqrt((((0.6 * 2 * bw * bw) ** 2 + (0.4 * d2[ok]) ** 2) * (EPS / unit[ok]) ** 2).mean())
    rms, rms_f32 = np.sqrt((err ** 2).mean()), max(np.sqrt((r ** 2).mean()) for r in ref)
    bias, bias_f32 = abs(err.mean()), max(abs(r.mean()) for r in ref)
    print(law, d, "rms", rms, "float32", rms_f32, "read", read, "mean", bias, bias_f32)
    pack = np.sqrt((((p2 - d2)[ok] / unit[ok]) ** 2).mean())
    assert rms <= 1.1 * np.sqrt(rms_f32 ** 2 + read ** 2 + pack ** 2)
    assert bias <= bias_f32 + 1.0


@pytest.mark.gpu
@pytest.mark.parametrize("l", [5, 300])
@pytest.mark.parametrize("n_z", [1, 64, 300])
def test_infinite_weights(l, n_z):
    """Infinite and NaN weights reach the results of their own labels only,
    an infinity as an infinity, by either form of the contraction."""
    n, d, bw = 128 * 300 + 5, 64, bw32(9.0)
    rng = np.random.default_rng(l + n_z)
    X = rng.standard_normal((n, d)).astype(np.float32)
    Z = rng.standard_normal((n_z, d)).astype(np.float32)
    a = rng.standard_normal((n, l)).astype(np.float32)
    a[31, 0], a[128 * 200 + 40, 1], a[n - 1, 2] = np.inf, -np.inf, np.nan
    a[5, l - 1], a[n // 2, l - 1] = np.inf, np.inf
    assert -(-n_z // 64) * 64 * n * d > 2 ** 27
    with Gpu(X, l, "gaussian", bw, 20, 2, np.arange(20)) as g:
        g.set_alpha(a)
        P = g.predict(Z)
    assert np.all(P[:, 0] == np.inf) and np.all(P[:, 1] == -np.inf)
    assert np.all(np.isnan(P[:, 2])) and np.all(P[:, l - 1] == np.inf)
    some = slice(3, 4)
    P_o = oracle.predict(X.astype(np.float64), a[:, some].astype(np.float64), Z.astype(np.float64),
                         oracle.GAUSSIAN, bw)
    assert np.max(np.abs(P[:, some] - P_o) / _bound(X, Z, a[:, some], "gaussian", bw)) <= 1.0
    assert np.all(np.isfinite(P[:, 3:l - 1]))


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", ["gaussian", "laplacian"])
def test_features_beyond_the_float32_squares(kernel):
    """Rows with an infinite or NaN feature, or whose squares overflow, give
    what the float32 expansion |x|^2 + |z|^2 - 2 x.z gives, with a NaN distance
    taken as 0: for queries and for centres."""
    n, d, n_z, bw = 128 * 300 + 5, 64, 130, bw32(9.0)
    rng = np.random.default_rng(3)
    X = rng.standard_normal((n, d)).astype(np.float32)
    Z = rng.standard_normal((n_z, d)).astype(np.float32)
    special = [np.inf, -np.inf, np.nan, np.float32(1e36), np.float32(-1e22)]
    for i, v in enumerate(special):
        Z[10 * i, 7] = v
        X[128 * 50 + 10 * i, 9] = v
    Z[60] = 1e25
    X[3000] = -1e25
    with np.errstate(all="ignore"):
        f = np.float32
        d2 = ((Z * Z).sum(1, dtype=f)[:, None] + (X * X).sum(1, dtype=f)[None]
              - f(2) * np.matmul(Z, X.T))
    odd_z = [10 * i for i in range(5)] + [60]
    odd_x = [128 * 50 + 10 * i for i in range(5)] + [3000]
    rows = np.setdiff1d(np.arange(n_z), odd_z)
    a = np.zeros((n, 8), dtype=np.float32)
    for j, c in enumerate(odd_x):            # the kernel values of the odd centres
        a[c, j] = 1.0
    a[rng.integers(0, n, 200), 6] = rng.standard_normal(200).astype(np.float32)
    a[odd_x, 6] = 0.0
    a[12345, 7] = 1.0
    with Gpu(X, 8, kernel, bw, 20, 2, np.arange(20)) as g:
        g.set_alpha(a)
        P = g.predict(Z)
    D = np.where(np.isnan(d2), 0.0, np.maximum(d2, 0.0)).astype(np.float64)
    K = np.exp(-D / (2 * bw * bw)) if kernel == "gaussian" else np.exp(-np.sqrt(D) / bw)
    want = K @ a.astype(np.float64)
    assert np.all(np.isfinite(P))
    # every value of an odd row or centre is 0 or 1 exactly
    assert np.array_equal(P[rows][:, :6], want[rows][:, :6])
    assert set(np.unique(want[rows][:, :6])) == {0.0, 1.0}
    assert np.array_equal(P[odd_z][:, 7], want[odd_z][:, 7])
    assert np.max(np.abs(P[odd_z][:, 6] - want[odd_z][:, 6])) < 1e-4
    ref = oracle.predict(X[a[:, 6] != 0].astype(np.float64), a[a[:, 6] != 0][:, 6:7].astype(np.float64),
                         Z[rows].astype(np.float64), kernel_id(kernel), bw)
    assert rel(P[rows][:, 6:7], ref) < TOL_STEP


# ---- the contraction's six products ------------------------------------------
#
# Distances of small integers are exact, so a kernel value is known to a few
# roundings, and with one nonzero weight to a label the result is one product:
# an error of 2^-17 in it, the size of the smallest of the six, shows.

CONTRACTIONS = [
    # l, n_z, ep_predict_noalloc (its kernel values come in several chunks
    # beyond 160 labels): one label tile to ten, queries shared by the waves or not
    (16, 1, False), (16, 100, False), (16, 300, False), (40, 40, False), (160, 30, False),
    (160, 300, False), (161, 20, False), (300, 300, False), (300, 300, True), (1100, 129, False),
]


def _contraction_problem(l):
    n, d = 128 * 300 + 5, 64
    rng = np.random.default_rng(l)
    X = rng.integers(-2, 3, (n, d)).astype(np.float32)
    X[128 * 7:128 * 8] = X[:128]             # (kernel values up to 1)
    at = (np.arange(l) * 9973 + 17) % n      # the centre of each label's weight
    w = (rng.uniform(1, 2, l) * np.exp2(rng.integers(-12, 13, l)) * rng.choice([-1, 1], l)).astype(np.float32)
    return n, d, X, at, w, bw32(10.0)


def _exact_kernel(X, Z, bw):
    scale = np.float64(np.float32(-np.log2(np.e) / (2 * bw * bw)))
    Xd, Zd = X.astype(np.float64), Z.astype(np.float64)
    d2 = (Zd ** 2).sum(1)[:, None] + (Xd ** 2).sum(1)[None] - 2 * Zd @ Xd.T
    return np.exp2(scale * d2)


# one product: the last addition truncated (2 eps), three products below 2^-26
# left out; a sum of five adds a rounding each
ONE, FIVE = 4 * EPS, 8 * EPS
# a kernel value: exp2 good to 2 eps, its argument (at most 4) rounded
VALUE = (2 + 4 * np.log(2) + 1) * EPS


@pytest.mark.gpu
@pytest.mark.parametrize("l,n_z,noalloc", CONTRACTIONS)
def test_every_product_of_the_contraction(l, n_z, noalloc):
    import paper_1806_06144_amd as ep
    n, d, X, at, w, bw = _contraction_problem(l)
    rng = np.random.default_rng(n_z)
    Z = X[rng.integers(0, n, n_z)].copy()
    Z[:, :40] = X[at[np.arange(n_z) % l], :40]
    assert -(-n_z // 64) * 64 * n * d > 2 ** 27

    with Gpu(X, l, "gaussian", bw, 20, 2, np.arange(20)) as g:
        def predict(a):
            g.set_alpha(a)
            out = g.torch.full((n_z, l), float("nan"), device=g.dev)
            call = ep.ep_predict_noalloc if noalloc else ep.ep_predict
            call(g.ctx, g.t(Z), n_z, out)
            ep.ep_sync(g.ctx)
            return out.cpu().numpy().astype(np.float64)

        a = np.zeros((n, l), dtype=np.float32)
        a[at, np.arange(l)] = 1.0
        K = predict(a)                       # head of the weight, all planes of the values
        K_o = _exact_kernel(X[at], Z, bw)
        assert K.max() > 0.3 and np.max(np.abs(K - K_o) / K_o) <= VALUE
        a[at, np.arange(l)] = w
        F = predict(a)
        assert np.max(np.abs(F - K * w) / (K * np.abs(w))) <= ONE
        # five centres of one group of 32 to a label
        a[:] = 0.0
        five = at[:, None] // 32 * 32 + (at[:, None] + 7 * np.arange(5)) % 32
        five = np.minimum(five, n - 1)
        ws = w[:, None] * np.float32([1.0, 0.3, -0.7, 0.11, 0.9])
        for i in range(5):
            np.add.at(a, (five[:, i], np.arange(l)), ws[:, i].astype(np.float32))
        F = predict(a)
    some = np.linspace(0, l - 1, min(l, 40)).astype(int)
    for j in some:
        rows = np.unique(five[j])
        Kj = _exact_kernel(X[rows], Z, bw)
        aj = a[rows, j].astype(np.float64)
        assert np.max(np.abs(F[:, j] - Kj @ aj) / (Kj @ np.abs(aj))) <= FIVE + VALUE


def _bf16(x):
    u = np.asarray(x, dtype=np.float32).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & np.uint32(0xFFFF0000)).view(np.float32)


@pytest.mark.parametrize("drop", [None] + [(i, j) for i in range(3) for j in range(3) if i + j <= 2])
def test_the_bound_shows_a_missing_product(drop):
    """The planes modelled in numpy: the bound above holds with the six
    products and fails with any one of them left out."""
    n, d, X, at, w, bw = _contraction_problem(161)
    Z = X[np.random.default_rng(1).integers(0, n, 200)]
    K = _exact_kernel(X[at], Z, bw).astype(np.float32)

    def planes(x):
        h = _bf16(x)
        m = _bf16(x - h)
        return h, m, _bf16(x - h - m)

    kp, wp = planes(K), planes(w)
    assert np.array_equal(kp[0] + kp[1] + kp[2], K) and np.array_equal(wp[0] + wp[1] + wp[2], w)
    F = sum(kp[j].astype(np.float64) * wp[i] for i in range(3) for j in range(3)
            if i + j <= 2 and (i, j) != drop)
    worst = np.max(np.abs(F - K.astype(np.float64) * w) / (K * np.abs(w).astype(np.float64)))
    assert (worst <= ONE) == (drop is None), worst / EPS


def _two_steps(n, d, l, s, k, m, kernel, bw, seed, batches=2):
    """Relative errors of f against float64 (on the device) over the first
    steps of a run, and S, the factor by which a step along the top eigenvector
    is larger than what steps 4-5 leave of it."""
    import torch
    import paper_1806_06144_amd as ep
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    X = torch.rand((n, d), device="cuda", generator=gen)
    X *= torch.rand((n, d), device="cuda", generator=gen) < 0.2
    perm = torch.randperm(n, device="cuda", generator=gen)
    r = perm[torch.randperm(n, device="cuda", generator=gen)[:s]]
    a = torch.randn((n, l), device="cuda", generator=gen) / n ** 0.5
    ctx, info = ep.ep_setup(X, n, d, l, kernel, bw, s, k, sub_idx=r.cpu().numpy())
    try:
        ep.ep_set_alpha(ctx, a)
        _, D, V, _ = ep.ep_get_preconditioner(ctx, info)
        D = torch.from_numpy(np.asarray(D)).cuda()
        V = torch.from_numpy(np.asarray(V).reshape(s, k)).cuda().double()

        def K64(p, q, i, j):
            x, y = X[i].double(), X[j].double()
            d2 = ((x * x).sum(1)[:, None] + (y * y).sum(1)[None]
                  - 2.0 * torch.matmul(x, y.T.contiguous())).clamp_(min=0.0)
            K = torch.exp(-d2 / (2 * bw * bw)) if kernel == "gaussian" else torch.exp(-d2.sqrt() / bw)
            K[i[:, None] == j[None, :]] = 1.0
            return K

        A = a.double()
        c = 1.0 / (info.beta + (m - 1) * info.lambda_k1)
        every, out, errs = torch.arange(n, device="cuda"), torch.empty((m, l), device="cuda"), []
        for b in range(batches):
            t = perm[b * m:(b + 1) * m].contiguous()
            y = torch.zeros((m, l), device="cuda")
            y[torch.arange(m), torch.randint(0, l, (m,), device="cuda", generator=gen)] = 1.0
            ep.ep_step(ctx, t, m, y, out)
            F = torch.matmul(K64(X, X, t, every), A)
            R = F - y.double()
            A[t] -= c * R
            G = torch.matmul(K64(X, X, r, t), R)
            A[r] += c * torch.matmul(V, D[:, None] * torch.matmul(V.T.contiguous(), G))
            ep.ep_sync(ctx)
            errs.append(float((out.double() - F).norm() / F.norm()))
    finally:
        ep.ep_destroy(ctx)
    return errs, m * c * info.sigma_1 / s


@pytest.mark.gpu
def test_second_step_keeps_its_precision():
    """From the second step of a run on, f is what steps 4-5 leave of a step
    along the top eigenvector that is S times larger, so the rounding of their
    sums shows S times as large: root mean square over shapes and runs at most
    1.5 * 2^-24 S. (The float32 pass with chunks of 256, and chunks of 64 summed
    in float32, are both at 2.0; with the chunks summed in float64 1.2.)"""
    e = []
    for s, m, k in [(4000, 520, 160), (4000, 1000, 160), (2000, 1001, 61)]:
        for seed in range(3):
            errs, S = _two_steps(20000, 784, 10, s, k, m, "gaussian", bw32(5.0), seed)
            e.append(errs[1] / (EPS * S))
    print("second step in units of 2^-24 S", e)
    assert np.sqrt(np.mean(np.square(e))) <= 1.5


# ---- which steps take the split pass -----------------------------------------

def _pass(g, m):
    import paper_1806_06144_amd as ep
    return {ep.EP_PASS_FLOAT32: "float32", ep.EP_PASS_SPLIT: "split",
            ep.EP_PASS_BLOCKED: "blocked"}[ep.ep_step_pass(g.ctx, m)]


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,d,l,ms", [
    # beyond 160 labels batches of more than 2048 rows keep the float32 pass
    ("gaussian", 700, 200, [(300, "split"), (2049, "float32"), (300, "split"), (2048, "split")]),
    ("gaussian", 700, 160, [(2049, "split"), (300, "split")]),
    # Laplacian steps do beyond 2048 features
    ("laplacian", 2049, 12, [(300, "float32"), (300, "float32")]),
    ("laplacian", 2048, 12, [(300, "split"), (300, "split")]),
    ("gaussian", 2049, 12, [(300, "split")]),
    # and passes of at most 2^27 multiply-adds
    ("gaussian", 699, 12, [(64, "split"), (30, "split")]), ("gaussian", 698, 12, [(64, "float32")]),
])
def test_steps_on_both_sides_of_a_line(kernel, d, l, ms):
    """Steps on one context that change pass, and predictions (always split
    here) between them, which read the planes of alpha that each step left."""
    n, s, k = 3001, 150, 12
    bw = bw32(1.3 if kernel == "gaussian" else 1.0)
    rng = np.random.default_rng(d + l)
    X = (rng.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
    Y = np.eye(l, dtype=np.float32)[rng.integers(0, l, n)]
    Z = (rng.standard_normal((400, d)) / np.sqrt(d)).astype(np.float32)
    a_o = a0 = (rng.standard_normal((n, l)) / np.sqrt(n)).astype(np.float32)
    r = rng.choice(n, s, replace=False)
    st = oracle.setup(X, kernel_id(kernel), bw, s, k, r)
    with Gpu(X, l, kernel, bw, s, k, r) as g:
        g.set_alpha(a0)
        for m, want in ms:
            assert _pass(g, m) == want
            t = rng.choice(n, m, replace=False)
            F = g.step(t, Y[t])
            a_o, F_o = oracle.step(st, a_o, t, Y[t])
            assert rel(F, F_o) < TOL_STEP
            P_o = oracle.predict(X.astype(np.float64), a_o, Z.astype(np.float64), kernel_id(kernel), bw)
            assert rel(g.predict(Z), P_o) < TOL_STEP
        assert rel(g.alpha() - a0, a_o - a0) < TOL_STEP
        # the form that is asked for: the float32 order stays reachable beyond 160 labels
        import paper_1806_06144_amd as ep
        ep.ep_set_contraction(g.ctx, "fused")
        gated = l > 160 or (kernel == "laplacian" and d > 2048)
        assert _pass(g, 300) == ("float32" if gated else "split")
        ep.ep_set_contraction(g.ctx, "blocked")
        assert (_pass(g, 300) == "blocked") == (d % 4 == 0)


@pytest.mark.gpu
@pytest.mark.parametrize("l", [6, 200])
@pytest.mark.parametrize("e", [-60, -50, -49, 40])
def test_features_scaled_by_a_power_of_two(e, l):
    """The same kernel values from features and bandwidth scaled by 2^e, down
    to rows whose squares are the smallest normal floats, where the rows share
    one scale (below 2^-49) and lo has 24 bits under the largest element."""
    n, d, n_z, bw = 128 * 300 + 5, 64, 70, 9.0
    rng = np.random.default_rng(1)
    X = rng.standard_normal((n, d)).astype(np.float32)
    Z = rng.standard_normal((n_z, d)).astype(np.float32)
    a = rng.standard_normal((n, l)).astype(np.float32)
    f = np.float32(2.0 ** e)
    P = []
    for s in (np.float32(1), f):
        with Gpu(X * s, l, "gaussian", float(np.float32(bw) * s), 20, 2, np.arange(20)) as g:
            g.set_alpha(a)
            P.append(g.predict(Z * s))
    # (the scaling is exact; below 2^-49 the low planes of small elements end
    # 2^-25 under the row's largest, a few roundings of the distance)
    assert rel(P[1], P[0]) < 1e-6
    P_o = oracle.predict(X.astype(np.float64), a.astype(np.float64), Z.astype(np.float64),
                         oracle.GAUSSIAN, bw)
    assert np.max(np.abs(P[1] - P_o) / _bound(X, Z, a, "gaussian", bw)) <= 1.0
