"""Moments of the basis refresh from many samples (the int8 matrix pipe): the edges of its tiles and panels, blocks that end a
basis or the gradient, scales that have to change on the way, whole numbers, numbers that are not finite."""
import numpy as np
import pytest

from paper_1811_03617_amd import gvq

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _fit(grads, M, d, cuts, dtype):
    b = gvq.Basis(M, d, 1, cuts, dtype)
    b.fit([g.to(DEV) for g in grads])
    C, n = b.export_cov()
    mu = b.export()[1]
    return b, C, n, mu


def _check(C, n, mu, grads, M, d, cuts):
    X = np.stack([g.to(torch.float64).numpy()[: M // d * d].reshape(-1, d) for g in grads])
    for i, (lo, hi) in enumerate(zip(cuts[:-1], cuts[1:])):
        x = X[:, lo:min(hi, M // d)].reshape(-1, d)
        assert n[i] == x.shape[0]
        m = x.mean(0)
        # as float64 sums of n products, with their n + 2 roundings at worst (test_every_digit and test_as_exact_products... look
        # closer)
        bound = (max(n[i], 64) + 4) * 2.0 ** -53 * (np.abs(x).T @ np.abs(x) / n[i] + 2 * np.outer(np.abs(m), np.abs(m)))
        assert np.all(np.abs(C[i] - (x.T @ x / n[i] - np.outer(m, m))) <= 2 * bound + 1e-300)
        assert np.array_equal(C[i], C[i].T)
        assert np.allclose(mu[i], m, rtol=1e-6, atol=1e-7 * np.abs(x).max())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [65, 79, 80, 81, 96, 97, 100, 112, 113, 127, 128, 129, 160, 161, 192, 193, 250, 385, 768, 1024])
def test_covariance_and_counts(d, dtype):
    rng = np.random.default_rng(d)
    L = 34 if d in (80, 128) else 5
    slices = 16384 // L + 147
    cuts = [0, slices - 75, slices - 74, slices] if d <= 300 else [0, slices]   # of one slice, and of a block and a few
    M = slices * d - (1 if d % 3 else 0)
    # columns of different size, samples that change their size on the way, columns that are zero at first or always
    size = 10.0 ** rng.uniform(-6, 0, d)
    grads = []
    for _ in range(L):
        x = rng.standard_normal((slices, d)) * size + 0.3 * size
        x[slices // 3: slices // 2] *= 1e-5
        x[slices // 2: slices // 2 + 200] = 0.0
        x[slices // 2 + 200: slices // 2 + 300] *= 1e3
        x[:100, 3] = 0.0
        x[:, d // 2] = 0.0
        grads.append(torch.from_numpy(x.reshape(-1)[:M].astype(np.float32)))
    if dtype == "bf16":
        grads = [g.to(torch.bfloat16) for g in grads]
    b, C, n, mu = _fit(grads, M, d, cuts if len(cuts) > 2 else None, dtype)
    b.close()
    _check(C, n, mu, grads, M, d, cuts)


# Numbers whose digits are known: a column's room is four times its largest number P, so that in units of 2^-47 of the room P is
# 2^45 and c = 100 (2^16 + 2^8) has 100 as its digits 3 and 4 (of 0 to 5), c + 100 as its digit 5 too.
_P, _C = 2 ** 45, 100 * (2 ** 16 + 2 ** 8)


def _digit_columns(d, slices, dtype):
    """P in every eighth sample of a column and its small number in the others; the sample's sign takes turns, so that the mean is
    0.  Returns the numbers (in units, float64) and sum x x^T over n samples of their kind as whole numbers, for multiples of 16."""
    small = np.full(d, _C)
    if dtype == "bf16":   # three digits hold nearly every number of a column: eight bits of digits 3 and 4, in few columns
        small[:] = 2 ** 37
        small[5::16] = 201 << 12
    else:
        small[5::16] += 100
    t, col = np.arange(16)[:, None], np.arange(d)[None, :]
    large = (t // 2 + col + col // 16) % 8 == 0   # elsewhere in the next columns, and in the next that have last digits
    x = np.where(large, _P, small).astype(object) * np.where(t % 2 == 0, 1, -1)
    gram = x.T.dot(x)
    assert slices % 16 == 0 and not x.sum(0).any()
    return np.tile(x.astype(np.float64), (slices // 16, 1)), gram * (slices // 16), small


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [65, 96, 112, 128, 144, 192])
def test_every_digit(d, dtype):
    """Every level of products that is to be there is: without the last one, or without the products of last digits, the sums are off by
    ten times the bound and more."""
    L, slices = 4, 4160
    x, gram, small = _digit_columns(d, slices, dtype)
    g = torch.from_numpy((x * 2.0 ** -45).astype(np.float32).reshape(-1))
    if dtype == "bf16":
        g = g.to(torch.bfloat16)
    assert np.array_equal(g.to(torch.float64).numpy(), (x * 2.0 ** -45).reshape(-1))
    b, C, n, mu = _fit([g] * L, slices * d, d, None, dtype)
    b.close()
    assert n[0] == L * slices and not mu.any()
    # in units: the ninth level and those below it are left out, 2^(-78 + 94) for a product of two digits, five such products of 100 x 100
    # and less at most, and 2^(-62 + 94) of every block and chunk where the eighth joins the seventh; then 2^-47 of the products'
    # absolute values for roundings (a chunk's Horner steps, 65 chunks, the quotient)
    left_out = slices * 5 * 1e4 * 2.0 ** 16 + (slices / 64 + 66) * 2.0 ** 32
    most = np.abs(x).T @ np.abs(x)
    off = np.abs((C[0] * 2.0 ** 90).astype(object) * slices - gram)
    assert np.all(off.astype(np.float64) <= left_out + most * 2.0 ** -47)


@pytest.mark.parametrize("d", [65, 128, 150])
def test_sums_that_fill_an_int(d):
    """More than a thousand blocks a task of digits -128: the sums of a level's products leave 32 bits unless they become float64 in
    between."""
    slices, L = 1 << 19, 32
    t, col = np.arange(8)[:, None], np.arange(d)[None, :]
    # -128 as digits 1, 2 and 3
    x = np.where((t + 3 * col) % 8 == 0, 1.0, -(2.0 ** -6) * (1 + 2.0 ** -8 + 2.0 ** -16)) * np.ones((8, d))
    g = torch.from_numpy(x.astype(np.float32)).to(DEV).repeat(slices // 8, 1).reshape(-1)
    assert np.array_equal(x, x.astype(np.float32))
    b = gvq.Basis(slices * d, d, 1, None, "f32")
    b.fit([g] * L)
    C, n = b.export_cov()
    b.close()
    m = x.mean(0)
    want = x.T @ x / 8 - np.outer(m, m)
    assert n[0] == slices * L
    # a chunk's few sums, up to 256 chunks in sixteen sums of sixteen, the covariance's three operations
    assert np.all(np.abs(C[0] - want) <= 2.0 ** -46 * (x.T @ x).max() / 8)


@pytest.mark.parametrize("scale", [2.0 ** -140, 2.0 ** -40, 1.0, 2.0 ** 40])
@pytest.mark.parametrize("d", [80, 128, 144])
def test_whole_numbers_are_exact(d, scale):
    rng = np.random.default_rng(d)
    L, slices = 3, 6000
    M = slices * d
    x = [rng.integers(-2000, 2001, M) for _ in range(L)]
    b, C, n, mu = _fit([torch.from_numpy((v * np.float64(scale)).astype(np.float32)) for v in x], M, d, None, "f32")
    b.close()
    X = np.concatenate([v.reshape(-1, d) for v in x])
    G, s = (X.T @ X).astype(np.float64), X.sum(0).astype(np.float64)   # below 2^53
    N = float(len(X))
    want = (G / N - np.outer(s / N, s / N)) * scale ** 2
    # a division, a product and a difference of exact sums
    assert np.all(np.abs(C[0] - want) <= 2.0 ** -51 * (G.max() / N + np.abs(np.outer(s, s)).max() / N ** 2) * scale ** 2)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("d", [128, 160])
def test_not_finite(d, bad):
    rng = np.random.default_rng(d)
    L, slices, column = 4, 5000, 17
    M = slices * d
    grads = [torch.from_numpy(rng.standard_normal(M).astype(np.float32)) for _ in range(L)]
    clean = [g.clone() for g in grads]
    grads[2][d * 1234 + column] = float(bad)
    b, C, n, mu = _fit(grads, M, d, None, "f32")
    with pytest.raises(gvq.GvqError) as e:
        b.fit_status()
    assert e.value.status == gvq.ENONFINITE
    b.close()
    assert not np.isfinite(C[0][column]).any() and not np.isfinite(mu[0][column])
    keep = np.arange(d) != column
    X = np.concatenate([g.to(torch.float64).numpy().reshape(-1, d) for g in clean])[:, keep]
    m = X.mean(0)
    assert np.allclose(C[0][np.ix_(keep, keep)], X.T @ X / len(X) - np.outer(m, m), rtol=0, atol=1e-12)


def test_same_bits_twice():
    rng = np.random.default_rng(3)
    d, slices, L = 200, 9000, 3
    grads = [torch.from_numpy(rng.standard_normal(slices * d).astype(np.float32)).to(DEV) for _ in range(L)]
    b = gvq.Basis(slices * d, d, 4)
    res = []
    for _ in range(2):
        b.fit(grads)
        res.append(b.export_cov()[0])
    b.close()
    assert np.array_equal(res[0], res[1])


def _gram(x):
    """sum x x^T: exact products, eight at a time in float64, the rest in long double."""
    total = np.zeros((x.shape[1],) * 2, np.longdouble)
    for i in range(0, len(x), 8):
        total += x[i:i + 8].T @ x[i:i + 8]
    return total


def _tails(name, slices, d, rng):
    x = rng.standard_normal((slices, d))
    if name == "lognormal":
        return np.exp(3.0 * x) * rng.choice([-1.0, 1.0], x.shape)
    if name == "one_sided":
        return np.exp(2.0 * x)
    if name == "fourth_power":
        return x ** 4
    if name == "few_large":
        return x * np.where(rng.random(x.shape) < 0.01, 1.0, 1e-3)
    if name == "two_sizes":
        return x * np.where(rng.random(x.shape) < 0.15, 1.0, 1e-6)
    if name == "some_tiny":
        return x * np.where(rng.random(x.shape) < 0.05, 1e-9, 1.0)
    if name == "constant_outliers":   # every column one number, with one large one, in another sample each
        x = np.repeat(np.abs(x[:1]) + 0.1, slices, 0)
        x[rng.integers(0, slices, d), np.arange(d)] *= 1000.0
        return x
    if name == "sizes_change":        # by blocks of samples, in both directions
        return x * 10.0 ** rng.uniform(-8, 0, slices // 64 + 1).repeat(64)[:slices, None]
    assert name == "student"
    return rng.standard_t(1.5, x.shape)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [65, 128, 192])
@pytest.mark.parametrize("name", ["lognormal", "one_sided", "fourth_power", "few_large", "two_sizes", "some_tiny",
                                  "constant_outliers", "sizes_change", "student"])
def test_as_exact_products_summed_in_float64(name, d, dtype):
    """Columns whose numbers differ in size by far more than a digit product holds: the sums have to be as good as float64 sums of
    exact products, relative to the sum of the products' absolute values."""
    rng = np.random.default_rng(d)
    L, slices = 4, 4200
    M = slices * d
    grads = [torch.from_numpy(_tails(name, slices, d, rng).astype(np.float32).reshape(-1)) for _ in range(L)]
    if dtype == "bf16":
        grads = [g.to(torch.bfloat16) for g in grads]
    b, C, n, mu = _fit(grads, M, d, None, dtype)
    b.close()
    x = np.concatenate([g.to(torch.float64).numpy().reshape(-1, d) for g in grads])
    N = len(x)
    assert n[0] == N
    G, m = _gram(x) / N, x.astype(np.longdouble).sum(0) / N
    most = np.abs(x).T @ np.abs(x) / N
    # Roundings one after the other: a sum of a chunk's samples (65 of each gradient or fewer) has no more than 4 * 65 of them,
    # that of the 65 chunks 65; the covariance is a quotient, a product and a difference behind it; 8 are the reference's.
    bound = (4 * 65 + 65 + 4 + 8) * 2.0 ** -53 * most + 2.0 ** -50 * np.abs(np.outer(m, m))
    assert np.all(np.abs(C[0] - (G - np.outer(m, m))) <= bound)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,B", [(65, 60), (112, 60), (128, 60), (161, 40), (250, 40)])
def test_long_tasks_that_change_pipes(d, B, dtype):
    """Bases of one chunk each, up to 300 blocks a task: heavy tails keep to the fp64 pipe for long, an outlier in every gradient takes
    a block or a few there, sizes that shrink for good leave it again.  A block lost, taken twice or mixed up is off by 1e-3."""
    rng = np.random.default_rng(d)
    L, lens = 34, 480 + 9 * (np.arange(B) % 13)
    cuts = [0] + [int(c) for c in lens.cumsum()]
    M = cuts[-1] * d - 1   # the last slice is not whole
    xs = []
    for g in range(3):
        x = rng.standard_normal((cuts[-1], d))
        for i in range(B):
            at = x[cuts[i]:cuts[i + 1]]
            if i % 3 == 0:
                at[:] = rng.standard_t(3, at.shape)
            elif i % 3 == 1:
                at[100 + 64 * g, d // 2] = 1e4
            else:
                at[200:] *= 1e-5 if g == 2 else 1.0
        xs.append(torch.from_numpy(x.astype(np.float32).reshape(-1)[:M]))
    if dtype == "bf16":
        xs = [x.to(torch.bfloat16) for x in xs]
    times = [20, 7, 7]   # the shrunken sizes come last
    b, C, n, mu = _fit([x for x, t in zip(xs, times) for _ in range(t)], M, d, cuts, dtype)
    b.close()
    X = [x.to(torch.float64).numpy()[: M // d * d].reshape(-1, d) for x in xs]
    for i, (lo, hi) in enumerate(zip(cuts[:-1], cuts[1:])):
        own = [x[lo:min(hi, M // d)] for x in X]
        assert n[i] == L * len(own[0])
        total = sum(t * (x.T @ x) for t, x in zip(times, own)) / n[i]
        most = sum(t * (np.abs(x).T @ np.abs(x)) for t, x in zip(times, own)) / n[i]
        m = sum(t * x.sum(0) for t, x in zip(times, own)) / n[i]
        # n roundings one after the other at worst, a few more for the covariance, as many again for the reference
        bound = (2 * n[i] + 16) * 2.0 ** -53 * (most + 2 * np.outer(np.abs(m), np.abs(m)))
        assert np.all(np.abs(C[i] - (total - np.outer(m, m))) <= bound)
        assert np.allclose(mu[i], m, rtol=1e-6, atol=1e-7 * max(np.abs(x).max() for x in own))
