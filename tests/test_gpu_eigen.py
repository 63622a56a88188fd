"""The eigensolver of the basis refresh at the edges of its kernels: matrix sizes around the register tiles of the
one-work-group tridiagonalisation (32, 64, 128), around the pieces of 64 that the long kernels hold per lane, odd sizes,
few and all eigenvectors; repeated eigenvalues and null spaces; sample counts around the 16 x 16 products of the
first-slice refresh.  Reference: numpy's symmetric eigensolver on the covariance that the library exports."""
import ctypes

import numpy as np
import pytest

from paper_1811_03617_amd import gvq

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _fit(slices, d, k, first_slice_only=False, dtype="f32"):
    """slices: list of [S][d] arrays, one per gradient."""
    b = gvq.Basis(slices[0].size, d, k, None, dtype)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    b.fit([torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32).reshape(-1)).to(DEV).to(tdt) for x in slices],
          first_slice_only=first_slice_only)
    status = b.fit_status()
    U, mu, eig = b.export()
    C, n = b.export_cov()
    b.close()
    return status, U[0].astype(np.float64), mu[0], eig[0], C[0], n[0]


def _check(U, eig, C, k, columns=None):
    d = C.shape[0]
    w = np.linalg.eigvalsh(C)[::-1]
    lam = w[0]
    # both solvers are backward stable: a few d roundings of the largest eigenvalue
    assert np.max(np.abs(eig - w)) <= 1e-15 * (d + 10) * lam
    assert np.all(np.diff(eig) <= 0)
    # U is rounded to fp32, each entry by at most 2^-24 of itself: products of two unit columns move by 2 * 2^-24,
    # C u - lambda u by at most (|C| + lambda) * 2^-24 |u| in 2-norm; 1e-8 for everything in float64
    assert np.max(np.abs(U.T @ U - np.eye(k))) <= 2 * 2.0 ** -24 + 1e-8
    cols = U[:, :columns]
    resid = np.linalg.norm(C @ cols - cols * eig[:cols.shape[1]], axis=0)
    assert np.max(resid) <= (2 * 2.0 ** -24 + 1e-8) * lam
    for i in range(k):
        assert U[np.argmax(np.abs(U[:, i])), i] > 0


@pytest.mark.parametrize("d,k", [(2, 1), (2, 2), (3, 2), (4, 4), (5, 1), (15, 15), (17, 4), (31, 31), (33, 9), (63, 63), (64, 64),
                                 (65, 17), (127, 127), (128, 128), (129, 129), (130, 1), (191, 33), (192, 64), (255, 65),
                                 (257, 31), (300, 300), (511, 32), (513, 100), (767, 96), (769, 128), (1023, 7), (1024, 130)])
def test_sizes(d, k):
    rng = np.random.default_rng(d * 1000 + k)
    A = rng.standard_normal((d, max(1, d // 8)))
    x = rng.standard_normal((2 * d + 70, A.shape[1])) @ A.T + 0.1 * rng.standard_normal((2 * d + 70, d))
    status, U, mu, eig, C, n = _fit([x], d, k)
    assert status > 0 and n == len(x)
    _check(U, eig, C, k)


@pytest.mark.parametrize("d,k", [(16, 16), (48, 20), (96, 96), (128, 40), (200, 80)])
@pytest.mark.parametrize("levels", [1, 3])
def test_repeated_eigenvalues(d, k, levels):
    """Slices +a_i e_i and -a_i e_i: C is diagonal with `levels` different entries, each many times over."""
    a = 1.0 + np.arange(d) % levels
    x = np.zeros((2 * d, d))
    x[np.arange(d), np.arange(d)] = a
    x[d + np.arange(d), np.arange(d)] = -a
    _, U, _, eig, C, _ = _fit([x], d, k)
    assert np.count_nonzero(C - np.diag(np.diag(C))) == 0
    _check(U, eig, C, k)


@pytest.mark.parametrize("d,k,rank", [(24, 24, 3), (64, 40, 5), (128, 60, 12), (160, 100, 9), (768, 96, 24)])
def test_more_columns_than_the_rank(d, k, rank):
    """Exactly rank-deficient data (small whole numbers): the trailing columns come from the null space."""
    rng = np.random.default_rng(d + rank)
    x = rng.integers(-3, 4, (3 * d, rank)).astype(np.float64) @ rng.integers(-2, 3, (rank, d))
    _, U, _, eig, C, _ = _fit([x], d, k)
    _check(U, eig, C, k)
    assert np.all(np.abs(eig[rank:]) <= 1e-12 * eig[0])


@pytest.mark.parametrize("d,k,L,dtype", [(64, 7, 2, "f32"), (65, 9, 3, "f32"), (96, 14, 15, "bf16"), (97, 15, 16, "f32"), (130, 16, 17, "f32"),
                                         (128, 31, 33, "f32"), (256, 60, 64, "bf16"), (257, 64, 65, "f32"), (768, 96, 100, "f32"),
                                         (1023, 127, 128, "f32"), (300, 50, 127, "f32"),     # the sample matrix
                                         (100, 30, 100, "f32"), (129, 20, 128, "f32"), (64, 64, 40, "bf16"),   # the covariance itself
                                         (768, 200, 20, "f32")])                             # most columns undetermined
def test_first_slice_sizes(d, k, L, dtype):
    rng = np.random.default_rng(d * 131 + L)
    x = [rng.standard_normal((3, d)) + 0.5 for _ in range(L)]
    if dtype == "bf16":
        x = [torch.from_numpy(v).to(torch.bfloat16).double().numpy() for v in x]
    else:
        x = [v.astype(np.float32).astype(np.float64) for v in x]
    _, U, mu, eig, C, n = _fit(x, d, k, first_slice_only=True, dtype=dtype)
    X = np.stack([v[0] for v in x])
    assert n == L
    np.testing.assert_allclose(mu, X.mean(0), rtol=2.0 ** -23, atol=1e-9)
    Xc = X - X.mean(0)
    assert np.max(np.abs(C - Xc.T @ Xc / L)) <= 1e-15 * (L + 10) * np.max(np.abs(C))
    assert np.array_equal(C, C.T)
    _check(U, eig, C, k, columns=min(k, L - 1))


@pytest.mark.parametrize("d,k", [(257, 257), (512, 288), (513, 289), (700, 320), (1000, 1000), (1024, 300)])
def test_many_columns(d, k):
    """More than 256 columns: panels finished in launches of their own, full and short last panels."""
    test_sizes(d, k)


@pytest.mark.parametrize("d,k,B", [(2, 2, 3000), (3, 1, 9000), (16, 5, 900), (16, 16, 5000), (33, 9, 600), (48, 20, 400), (64, 64, 300),
                                   (65, 30, 300), (128, 16, 600), (40, 12, 120)])
def test_many_small_matrices(d, k, B):
    """Bases side by side, for every number of lanes that shares an eigenvalue (16, 8 and 4 from 4096, 16384 and 32768 rows of
    matrices on), matrices with few rows in a part of a work-group, a zero matrix and unequal scales among them."""
    rng = np.random.default_rng(d * B)
    per = d + 9 + rng.integers(0, 5, B)
    cuts = np.concatenate([[0], np.cumsum(per)])
    x = rng.standard_normal((cuts[-1], d)) * np.exp(rng.uniform(-6, 6, B)).repeat(per)[:, None]
    x[cuts[7]:cuts[8]] = 0.25
    b = gvq.Basis(x.size, d, k, cuts, "f32")
    b.fit([torch.from_numpy(x.astype(np.float32).reshape(-1)).to(DEV)])
    assert b.fit_status() > 0
    U, mu, eig = b.export()
    C, n = b.export_cov()
    b.close()
    assert np.array_equal(n, per)
    w = np.linalg.eigvalsh(C)[:, ::-1]
    lam = w[:, :1]
    assert not C[7].any() and not eig[7].any() and np.array_equal(U[7], np.eye(d, k))
    assert np.all(np.abs(eig - w) <= 1e-15 * (d + 10) * lam)
    U = U.astype(np.float64)
    assert np.max(np.abs(np.swapaxes(U, 1, 2) @ U - np.eye(k))) <= 2 * 2.0 ** -24 + 1e-8
    resid = np.linalg.norm(C @ U - U * eig[:, None, :k], axis=1)
    assert np.all(resid <= (2 * 2.0 ** -24 + 1e-8) * lam)


def test_status_reports_what_the_solver_did():
    """The most solves for any vector: at least two where there was something to solve, none for a zero covariance, whatever
    the handle's last fit left behind."""
    d, k = 24, 5
    rng = np.random.default_rng(5)
    x = torch.from_numpy(rng.standard_normal(50 * d).astype(np.float32)).to(DEV)
    bad = x.clone()
    bad[7] = float("nan")
    b = gvq.Basis(x.numel(), d, k)
    for first_slice_only in (False, True):
        grads = [x, x.roll(11), x.roll(30)]
        b.fit(grads, first_slice_only=first_slice_only)
        assert 2 <= b.fit_status() <= 5
        b.fit([torch.ones_like(x)] * 3, first_slice_only=first_slice_only)
        assert b.fit_status() == 0
        b.fit([x, bad, x], first_slice_only=first_slice_only)
        with pytest.raises(gvq.GvqError) as e:
            b.fit_status()
        assert e.value.status == gvq.ENONFINITE
    b.fit(grads)
    assert 2 <= b.fit_status() <= 5
    b.close()


@pytest.mark.parametrize("d,k,B", [(136, 9, 2), (137, 9, 14), (137, 9, 15), (300, 40, 6), (300, 40, 7), (1024, 5, 2), (1024, 5, 3)])
def test_matrices_that_share_the_chip(d, k, B):
    """Bases side by side on both sides of where their rows no longer fit the compute units together (256 groups of 8 rows)."""
    rng = np.random.default_rng(d * B)
    per = 2 * d + 11
    x = (rng.standard_normal((B * per, d // 8)) @ rng.standard_normal((d // 8, d))
         + 0.1 * rng.standard_normal((B * per, d))) * np.exp(rng.uniform(-6, 6, B)).repeat(per)[:, None]
    if B > 2:
        x[per:2 * per] = 0.25
    b = gvq.Basis(x.size, d, k, np.arange(B + 1) * per, "f32")
    g = torch.from_numpy(x.astype(np.float32).reshape(-1)).to(DEV)
    for _ in range(2):   # also what the fit before left behind
        b.fit([g])
        assert b.fit_status() > 0
    U, _, eig = b.export()
    C, _ = b.export_cov()
    b.close()
    for i in range(B):
        if B > 2 and i == 1:
            assert not eig[i].any() and np.array_equal(U[i], np.eye(d, k))
        else:
            _check(U[i].astype(np.float64), eig[i], C[i], k)


def test_refreshes_on_several_streams_and_captured():
    """Handles refreshed on streams of their own at the same time give the bits of one after the other, and so does a captured
    refresh at every replay."""
    n, d, k = 4, 520, 24
    rng = np.random.default_rng(3)
    xs = [torch.from_numpy((rng.standard_normal((900, 40)) @ rng.standard_normal((40, d))
                            + 0.1 * rng.standard_normal((900, d))).astype(np.float32).reshape(-1)).to(DEV) for _ in range(n)]
    bases = [gvq.Basis(900 * d, d, k) for _ in range(n)]
    alone = []
    for b, x in zip(bases, xs):
        b.fit([x])
        b.fit_status()
        alone.append(b.export())
    streams = [torch.cuda.Stream() for _ in range(n)]
    torch.cuda.synchronize()
    for _ in range(3):
        for b, x, s in zip(bases, xs, streams):
            b.fit([x], stream=s.cuda_stream)
    torch.cuda.synchronize()
    for b, want in zip(bases, alone):
        for got, w in zip(b.export(), want):
            assert np.array_equal(got, w)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=streams[0]):
        bases[0].fit([xs[0]], stream=streams[0].cuda_stream)
    for _ in range(3):
        bases[0].fit([xs[1]])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert bases[0].fit_status() > 0
        for got, w in zip(bases[0].export(), alone[0]):
            assert np.array_equal(got, w)
        C, _ = bases[0].export_cov()
        _check(alone[0][0][0].astype(np.float64), alone[0][2][0], C[0], k)
    for b in bases:
        b.close()


@pytest.mark.parametrize("d,k", [(129, 3), (136, 136), (255, 20), (257, 20), (512, 30), (513, 30), (700, 7), (768, 96), (769, 9), (1024, 40)])
def test_captured_refresh_has_the_bits_of_an_eager_one(d, k):
    """Above 128 rows an eager refresh reduces the matrix in one launch, a captured one column by column."""
    gen = torch.Generator(device=DEV).manual_seed(d)
    x = torch.randn(d + 60, 50, generator=gen, device=DEV) @ torch.randn(50, d, generator=gen, device=DEV)
    x = (x + 0.1 * torch.randn(d + 60, d, generator=gen, device=DEV)).reshape(-1)
    b = gvq.Basis(x.numel(), d, k)
    b.fit([x])
    b.fit_status()
    eager = b.export()
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        b.fit([x], stream=stream.cuda_stream)
    for _ in range(2):
        b.import_(np.zeros((1, d, k), np.float32), np.zeros((1, d), np.float32))
        graph.replay()
        torch.cuda.synchronize()
        for got, want in zip(b.export(), eager):
            assert np.array_equal(got, want)
    b.close()


def _hip():
    """The HIP runtime that PyTorch has loaded, for what PyTorch has no call for."""
    torch.cuda.init()
    with open("/proc/self/maps") as maps:
        return ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64" in line))


@pytest.mark.parametrize("d,k,B", [(300, 40, 6), (768, 96, 1), (1024, 5, 2)])
@pytest.mark.parametrize("units", [(0xFFFFFFFF,) + (0,) * 7, (0x0000FFFF,) * 8, (0xFFFFFFFF,) * 7 + (0x7FFFFFFF,)])
def test_refresh_on_a_stream_with_few_compute_units(d, k, B, units):
    """The work-groups of a matrix that do not have the chip to themselves must not wait for each other."""
    gen = torch.Generator(device=DEV).manual_seed(d)
    x = torch.randn(B * (d + 9), d, generator=gen, device=DEV).reshape(-1)
    b = gvq.Basis(x.numel(), d, k, [i * (d + 9) for i in range(B + 1)])
    b.fit([x])
    b.fit_status()
    want = b.export()
    hip, stream = _hip(), ctypes.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 8, (ctypes.c_uint32 * 8)(*units)) == 0
    b.import_(np.zeros((B, d, k), np.float32), np.zeros((B, d), np.float32))
    b.fit([x], stream=stream.value)
    assert b.fit_status(stream=stream.value) >= 2
    for got, w in zip(b.export(), want):
        assert np.array_equal(got, w)
    b.close()
    assert hip.hipStreamDestroy(stream) == 0


@pytest.mark.parametrize("d,k,B", [(129, 129, 1), (136, 9, 14), (257, 20, 3), (520, 24, 1), (768, 96, 1), (1024, 5, 2)])
def test_refresh_whose_work_groups_stop_waiting(d, k, B):
    """Option 6: the one launch gives up at the first word that has not arrived, and the columns are done over one by one: the
    bits of the undisturbed refresh, many times its time (which shows that the launch did give up).  One basis is constant."""
    gen = torch.Generator(device=DEV).manual_seed(d)
    x = torch.randn(B, d + 9, d, generator=gen, device=DEV)
    if B > 2:
        x[1] = 0.5
    x = x.reshape(-1)
    b = gvq.Basis(x.numel(), d, k, [i * (d + 9) for i in range(B + 1)])

    def refresh():
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        b.fit([x])
        end.record()
        solves = b.fit_status()
        return solves, start.elapsed_time(end), b.export()

    refresh()
    solves, usual, want = refresh()
    for polls in (1, 0):
        try:
            gvq.gvq_set_option(6, polls)
            got = refresh()
        finally:
            gvq.gvq_set_option(6, 0)
        print(d, B, polls, usual, got[1])
        assert got[0] == solves
        for a, w in zip(got[2], want):
            assert np.array_equal(a, w)
        if polls and d > 200:
            assert got[1] > 2 * usual
    b.close()


class _Busy:
    """A stream with a long, finite queue: copies that take about a quarter of a second."""

    def __init__(self):
        self.x = torch.empty(1 << 28, device=DEV)   # 1 GiB, about 0.35 ms a copy
        self.y = torch.empty_like(self.x)
        self.stream, self.done = torch.cuda.Stream(), torch.cuda.Event()

    def start(self):
        torch.cuda.synchronize()
        with torch.cuda.stream(self.stream):
            for _ in range(700):
                self.y.copy_(self.x)

    def end(self):
        self.done.record(self.stream)


def test_status_waits_for_its_own_stream_only():
    """Another stream still has work when the answer is there (one of several streams: two may share a hardware queue)."""
    x = torch.randn(64 * 500, device=DEV)
    b = gvq.Basis(64 * 500, 64, 8)
    b.fit([x])
    solves = b.fit_status()
    busy = _Busy()
    streams = [torch.cuda.Stream() for _ in range(3)]
    busy.start()
    busy.end()
    early = 0
    for s in streams:
        assert b.fit_status(stream=s.cuda_stream) == solves
        early += not busy.done.query()
    torch.cuda.synchronize()
    assert early
    b.close()


def test_refresh_does_not_wait_for_another_stream():
    """A refresh above 128 elements that is queued behind long work on one stream does not hold up a refresh on another, nor the
    next one on its own stream; all have the bits of one done alone."""
    n, d, k = 5, 520, 24
    gen = torch.Generator(device=DEV).manual_seed(6)
    xs = [torch.randn(600 * d, generator=gen, device=DEV) for _ in range(n)]
    bases = [gvq.Basis(600 * d, d, k) for _ in range(n)]
    alone = []
    for b, x in zip(bases, xs):
        b.fit([x])
        b.fit_status()
        alone.append(b.export())
    busy = _Busy()
    streams = [torch.cuda.Stream() for _ in range(n - 2)]
    busy.start()
    for b, x in zip(bases[:2], xs):
        b.fit([x], stream=busy.stream.cuda_stream)
    busy.end()
    early = 0
    for b, x, s in zip(bases[2:], xs[2:], streams):   # several: two may share a hardware queue
        b.fit([x], stream=s.cuda_stream)
        assert b.fit_status(stream=s.cuda_stream) >= 2
        early += not busy.done.query()
    torch.cuda.synchronize()
    assert early
    for b, want in zip(bases, alone):
        for got, w in zip(b.export(), want):
            assert np.array_equal(got, w)
        b.close()
