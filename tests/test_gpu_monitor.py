"""Parity of gvq_local_loss (Eq. 6) and gvq_select_k (Eq. 5) with the float64 oracle."""
import numpy as np
import pytest

import oracle
from paper_1811_03617_amd import Workload, gvq, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _wl(M, d, k, N, dtype="f32", rank=3, block_elems=0, seed=5, L=2, sigma=0.2):
    return Workload("t", M, d, k, N, L, dtype, rank, sigma, block_elems=block_elems, seed=seed)


def _check_loss(w, mean_offset=None):
    offs = w.block_offsets()
    if w.M < w.d:   # no full slice to fit on: any orthonormal basis serves
        rng = np.random.default_rng(w.seed)
        U = np.linalg.qr(rng.standard_normal((w.d, w.k)))[0][None]
        mu = rng.standard_normal((1, w.d))
    else:
        fit_np = [synth.to_numpy(g) for g in synth.fit_gradients(w, "cpu", mean_offset=mean_offset)]
        U, mu, _ = oracle.fit(fit_np, w.d, w.k, dtype=w.dtype, offsets=offs)
    U32, mu32 = U.astype(np.float32), mu.astype(np.float32)
    U64, mu64 = U32.astype(np.float64), mu32.astype(np.float64)
    workers = synth.worker_gradients(w, "cpu", mean_offset=mean_offset)
    b = gvq.Basis(w.M, w.d, w.k, offs, w.dtype)
    b.import_(U32, mu32)
    out = torch.full((w.n_blocks,), float("nan"), device=DEV, dtype=torch.float64)
    for g in workers[:2]:
        gh = synth.to_numpy(g)
        ref = oracle.local_loss(gh, U64, mu64, w.N, dtype=w.dtype, offsets=offs)
        b.local_loss(g.to(DEV), w.N, out)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        # energy of the centred gradient per basis: the scale rounding noise is relative to
        Uz = np.zeros((w.n_blocks, w.d, 1))
        energy = oracle.local_loss(gh, Uz, mu64, w.N, dtype=w.dtype, offsets=offs)
        assert np.all(np.isfinite(got))
        assert np.all(np.abs(got - ref) <= 1e-4 * ref + 1e-9 * energy), (got, ref)
        # second call gives the same bits (fixed summation order)
        out2 = torch.empty_like(out)
        b.local_loss(g.to(DEV), w.N, out2)
        torch.cuda.synchronize()
        assert torch.equal(out, out2)
    b.close()


@pytest.mark.parametrize("M,d,k,N", [
    (16 * 1000 + 5, 16, 4, 4), (32 * 2111 + 8, 32, 8, 8), (64 * 1777 + 40, 64, 16, 8),
    (128 * 1531 + 40, 128, 32, 16), (128 * 777 + 127, 128, 16, 3), (128 * 200 + 3, 128, 7, 2),
    (64 * 300 + 1, 64, 32, 2), (32 * 500 + 31, 32, 32, 2), (100, 128, 32, 2),
])
def test_local_loss_mfma_shapes(M, d, k, N):
    _check_loss(_wl(M, d, k, N))


@pytest.mark.parametrize("M,d,k,N", [(24 * 501 + 5, 24, 5, 3), (2 * 1000 + 1, 2, 1, 2),
                                      (100 * 77 + 60, 100, 100, 2), (128 * 65 + 9, 128, 40, 2)])
def test_local_loss_generic_shapes(M, d, k, N):
    _check_loss(_wl(M, d, k, N, rank=1 if d < 4 else 3))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_local_loss_many_bases_and_mean(dtype):
    _check_loss(_wl(128 * 1000 + 40, 128, 16, 4, dtype=dtype, block_elems=128 * 77),
                mean_offset=np.linspace(-3, 5, 128))
    _check_loss(_wl(32 * 4000 + 8, 32, 8, 2, dtype=dtype, block_elems=32 * 1000))
    _check_loss(_wl(24 * 400 + 3, 24, 6, 2, dtype=dtype, block_elems=24 * 50))


def test_local_loss_error_paths():
    L = gvq.lib()
    b = gvq.Basis(16 * 100, 16, 4)
    x = torch.zeros(16 * 100, device=DEV)
    o = torch.zeros(2, device=DEV, dtype=torch.float64)
    st = torch.cuda.current_stream().cuda_stream
    assert L.gvq_local_loss(b.handle, x.data_ptr(), 1, o.data_ptr(), st) == gvq.ENOTFIT
    b.import_(np.zeros((1, 16, 4), np.float32), np.zeros((1, 16), np.float32))
    assert L.gvq_local_loss(b.handle, x.data_ptr(), 0, o.data_ptr(), st) == gvq.EINVAL
    assert L.gvq_local_loss(b.handle, x.data_ptr() + 4, 1, o.data_ptr(), st) == gvq.EALIGN
    assert L.gvq_local_loss(b.handle, x.data_ptr(), 1, o.data_ptr() + 4, st) == gvq.EALIGN
    assert L.gvq_local_loss(b.handle, x.data_ptr(), 1, None, st) == gvq.EINVAL
    b.close()


@pytest.mark.parametrize("M,d,k,block_elems", [(64 * 3000, 64, 16, 0), (16 * 5000, 16, 4, 0),
                                                (128 * 900 + 40, 128, 16, 128 * 100), (24 * 1000, 24, 5, 0)])
def test_select_k_matches_the_oracle(M, d, k, block_elems):
    import ctypes as C
    w = _wl(M, d, k, 2, rank=5 if d > 8 else 2, block_elems=block_elems, L=3)
    offs = w.block_offsets()
    fit = synth.fit_gradients(w, "cpu")
    _, _, eig_o = oracle.fit([synth.to_numpy(g) for g in fit], d, k, offsets=offs)
    b = gvq.Basis(M, d, k, offs)
    st = torch.cuda.current_stream().cuda_stream
    out = (C.c_int * w.n_blocks)()
    assert gvq.lib().gvq_select_k(b.handle, 0.01, out, st) == gvq.ENOTFIT
    b.fit([g.to(DEV) for g in fit])
    _, _, eig = b.export()
    for lam in (0.5, 0.1, 0.01, 1e-3, 1e-5, 0.0):
        got = b.select_k(lam)
        want = oracle.select_k(eig_o, lam)
        for bb in range(w.n_blocks):
            if eig[bb].sum() <= 0:      # a basis without samples: nothing to lose
                assert got[bb] == 1 and want[bb] == 1
                continue
            frac = np.cumsum(eig[bb]) / eig[bb].sum()
            if got[bb] != want[bb]:   # only possible when the ratio sits on the threshold
                assert abs(frac[min(got[bb], want[bb]) - 1] - (1 - lam)) < 1e-10
            assert frac[got[bb] - 1] >= 1 - lam - 1e-12
            assert got[bb] == 1 or frac[got[bb] - 2] < 1 - lam + 1e-12
    assert gvq.lib().gvq_select_k(b.handle, 1.0, out, st) == gvq.EINVAL
    assert gvq.lib().gvq_select_k(b.handle, -0.1, out, st) == gvq.EINVAL
    b.close()


@pytest.mark.parametrize("d,k", [(64, 17), (64, 32), (128, 17), (128, 21), (128, 32)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_local_loss_three_term_products(d, k, dtype):
    """One basis, 17 to 32 comps: sizes around the 16-slice tiles and the runs of 2048 elements, every wave with several runs, and
    the bounds-checked tiles alone; float64 for reference.  A residual element carries the rounding of sums of d and k products,
    at most (d + k) 2^-24 |x| each, half of that at random: relative to the loss r^2 that is 2 (d + k) 2^-25 |x| / r at most."""
    rng = np.random.default_rng(d + k)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    U = np.linalg.qr(rng.standard_normal((d, k)))[0].astype(np.float32)
    mu = rng.standard_normal(d).astype(np.float32)
    U64, mu64 = torch.from_numpy(U).to(DEV).double(), torch.from_numpy(mu).to(DEV).double()
    gen = torch.Generator(device=DEV).manual_seed(d)
    for M in (1, d - 1, d, 16 * d - 1, 16 * d, 2047, 2048, 2049, 2048 + 16 * d + 5, 64 * 2048, 131 * 2048 + 17 * d + 3, 9000 * 2048 + 1):
        S = -(-M // d)
        z = torch.randn(S, k, generator=gen, device=DEV, dtype=torch.float64)
        x = (z @ U64.T + 0.05 * torch.randn(S, d, generator=gen, device=DEV, dtype=torch.float64) + mu64 / 3).reshape(-1)[:M].to(tdt)
        b = gvq.Basis(M, d, k, None, dtype)
        b.import_(U, mu)
        out = torch.empty(1, device=DEV, dtype=torch.float64)
        whole = torch.zeros(S * d, device=DEV, dtype=torch.float64)
        whole[:M] = x.double()
        c = whole.view(S, d) - mu64 / 3
        r = (c - (c @ U64) @ U64.T).reshape(-1)[:M]
        want, size = float(r @ r), float((c * c).sum())
        for mask in ((0, 1) if M < 1 << 20 else (0,)):
            try:
                gvq.gvq_set_option(3, mask)
                b.local_loss(x, 3, out)
            finally:
                gvq.gvq_set_option(3, 0)
            assert abs(float(out) - want) <= (d + k) * 2.0 ** -24 * (want * size) ** 0.5, (M, mask)
        b.close()


@pytest.mark.parametrize("scale", [0.0, 1e-18, 1e17, 3.4e38])
def test_local_loss_three_term_products_at_the_ends_of_the_range(scale):
    """Numbers that round up to infinity in bf16 stay finite terms: the loss is finite or overflows as the sum of squares does."""
    d, k, S = 128, 32, 40
    rng = np.random.default_rng(1)
    U = np.linalg.qr(rng.standard_normal((d, k)))[0].astype(np.float32)
    x = (rng.uniform(0.25, 0.9999, (S, d)) * scale).astype(np.float32)
    if scale > 1e30:   # sums of many such numbers overflow in fp32 whatever the products; |U^T x| <= |x| of one does not
        x[:, 1:] = 0
    b = gvq.Basis(S * d, d, k)
    b.import_(U, np.zeros(d, np.float32))
    out = torch.empty(1, device=DEV, dtype=torch.float64)
    b.local_loss(torch.from_numpy(x).to(DEV).reshape(-1), 1, out)
    r = x.astype(np.float64) @ (np.eye(d) - U.astype(np.float64) @ U.T.astype(np.float64))
    want = float((r * r).sum())
    if scale < 1e30:
        assert abs(float(out) - want) <= 1e-5 * want   # (d + k) 2^-24, |x| of the order of the residual
    else:
        assert float(out) == float("inf")              # squares of fp32 residuals overflow
    for bad in (float("nan"), float("inf")):
        x[3, 5] = bad
        b.local_loss(torch.from_numpy(x).to(DEV).reshape(-1), 1, out)
        assert np.isnan(float(out))
    b.close()


def _bf16_terms(v, nearest):
    """fp32 numbers as three bf16 terms, each what the ones before leave, cut off or rounded to nearest even."""
    terms, rest = [], v.astype(np.float32)
    for _ in range(3):
        bits = rest.view(np.uint32)
        if nearest:
            bits = bits + (0x7FFF + ((bits >> 16) & 1)).astype(np.uint32)
        t = (bits & np.uint32(0xFFFF0000)).view(np.float32)
        terms.append(t.astype(np.float64))
        rest = rest - t
    return terms


def _emulated_residual(c, U, first=(), second=()):
    """|c - U U^T c| with both products made of terms, i + j <= 2 but for the pairs named; sums in float64."""
    def product(a, b, dropped):
        return sum(a[i] @ b[j] for i in range(3) for j in range(3 - i) if (i, j) not in dropped)
    u = _bf16_terms(U, True)
    y = product(_bf16_terms(c, False), u, first).astype(np.float32)
    return np.linalg.norm(c.astype(np.float64) - product(_bf16_terms(y, False), [t.T for t in u], second))


@pytest.mark.parametrize("d,k", [(64, 17), (64, 32), (128, 17), (128, 21), (128, 32)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_local_loss_keeps_all_six_products(d, k, dtype):
    """Slices that lie in the span of U but for the rounding of their elements: the residual is what the arithmetic leaves.  It is r + e,
    e: the roundings of fp32 sums (6 d / 32 + 6 products of 32 terms each, at random: their root, 7 at most, times 2^-25),
    of c = x - mu / N (2^-25 of |c| and |mu| / N each) and the products that are left out (3 * 2^-24 at most), so | |r + e| - |r| | <=
    8 * 2^-24 |c|.  Leaving out any one of the six products of either contraction gives more, as the emulation shows here."""
    rng = np.random.default_rng(d + k)
    U = np.linalg.qr(rng.standard_normal((d, k)))[0].astype(np.float32)
    U64 = U.astype(np.float64)
    bound, worst, seen = 8 * 2.0 ** -24, 0.0, {}
    for S in (5, 16, 37, 64 * 2048 // d, 131 * 2048 // d + 17, 3000 * 2048 // d + 1):
        n = min(S, 400)
        if dtype == "f32":
            mu = rng.standard_normal(d).astype(np.float32)
            x = (rng.standard_normal((n, k)) @ U64.T + mu / 3.0).astype(np.float32)
        else:   # one slice; the mean makes up for its rounding to bf16
            v = rng.standard_normal((1, k)) @ U64.T
            x = (v.astype(np.float32).view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
            mu = (3.0 * (x - v)).astype(np.float32)[0]
        x = x[np.arange(S) % len(x)]
        c = x[:n].astype(np.float64) - mu.astype(np.float64) / 3
        times = np.bincount(np.arange(S) % n, minlength=n)
        want = np.sqrt(times @ np.sum((c - (c @ U64) @ U64.T) ** 2, axis=1))
        size = np.sqrt(times @ np.sum(c ** 2, axis=1))
        b = gvq.Basis(S * d, d, k, None, dtype)
        b.import_(U, mu)
        g = torch.from_numpy(x.reshape(-1)).to(DEV).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
        out = torch.empty(1, device=DEV, dtype=torch.float64)
        for mask in (0, 1):
            try:
                gvq.gvq_set_option(3, mask)
                b.local_loss(g, 3, out)
            finally:
                gvq.gvq_set_option(3, 0)
            err = abs(float(out) ** 0.5 - want) / size
            worst = max(worst, err)
            assert err <= bound, (S, mask, err * 2 ** 24)
        b.close()
        c32 = c.astype(np.float32)
        r, size = np.linalg.norm(c - (c @ U64) @ U64.T), np.linalg.norm(c)
        assert abs(_emulated_residual(c32, U) - r) <= bound * size / 4
        for pair in ((0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)):
            for which in ("first", "second"):
                lost = abs(_emulated_residual(c32, U, **{which: (pair,)}) - r) / size
                seen[which, pair] = max(seen.get((which, pair), 0.0), lost)
    print(d, k, dtype, "worst", worst * 2 ** 24, "least lost", min(seen.values()) * 2 ** 24)
    assert min(seen.values()) > bound
