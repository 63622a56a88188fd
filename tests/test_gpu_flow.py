"""Eqs. (2) and (4) on the slice lengths and comps that no other kernel is made for: lengths and comps around the multiples of
4, 16 and 32 where a word, a tile or a contraction step is left over, one and several bases, ranges that start and end inside
a tile, the fused ring step, both storage types, against float64 and against the LDS-tiled kernels."""
import numpy as np
import pytest

from paper_1811_03617_amd import gvq

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [(4, 1), (4, 4), (5, 2), (7, 3), (12, 5), (13, 3), (16, 16), (17, 4), (24, 6), (31, 9), (33, 11), (48, 12), (63, 30),
          (65, 16), (77, 19), (96, 33), (100, 25), (127, 42), (128, 43), (128, 128), (129, 17), (160, 80), (193, 64), (201, 50),
          (255, 31), (257, 86), (300, 100), (321, 128), (385, 48), (400, 111), (500, 62), (513, 128), (601, 20), (640, 106),
          (700, 97), (767, 128), (768, 7)]


def _make(d, k, dtype, cuts, M, rng):
    S = -(-M // d)
    B = 1 if cuts is None else len(cuts) - 1
    U = np.stack([np.linalg.qr(rng.standard_normal((d, k)))[0] for _ in range(B)]).astype(np.float32)
    mu = (0.3 * rng.standard_normal((B, d))).astype(np.float32)
    b = gvq.Basis(M, d, k, cuts, dtype)
    b.import_(U, mu)
    g = torch.from_numpy(rng.standard_normal(M).astype(np.float32))
    if dtype == "bf16":
        g = g.to(torch.bfloat16)
    which = np.zeros(S, dtype=np.int64) if cuts is None else np.searchsorted(np.array(cuts), np.arange(S), side="right") - 1
    x = np.zeros(S * d)
    x[:M] = g.to(torch.float64).numpy()
    return b, g.to(DEV), U.astype(np.float64)[which], mu.astype(np.float64)[which], x.reshape(S, d)


def _close(got, want, tol, what):
    # tol: of the largest value; d or k fp32 roundings in the exact kernels, 2^-17 a product in the split ones
    assert np.all(np.isfinite(got)), what
    err = np.max(np.abs(got - want)) / np.max(np.abs(want))
    assert err <= tol, f"{what}: {err:.2e}"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("blocks", [1, 3])
@pytest.mark.parametrize("d,k", SHAPES)
def test_matches_float64_and_the_general_route(d, k, blocks, dtype):
    rng = np.random.default_rng(1000 * d + k)
    slices = max(200, 40_000 // d) + 3
    M = slices * d - (d // 3 if d > 4 else 0)
    cuts = None if blocks == 1 else [0, slices // 3 + 1, slices // 3 + 2, slices]
    b, g, U, mu, x = _make(d, k, dtype, cuts, M, rng)
    exact = 2.0 * d * k / (4.0 * (d + k)) < 10.0
    tol = 2e-6 if exact else 4e-5
    N = 3
    y = torch.empty(slices * k, device=DEV)
    y.fill_(float("nan"))
    b.compress(g, N, y)
    want = np.einsum("sdk,sd->sk", U, x - mu / N)
    _close(y.cpu().numpy().reshape(slices, k), want, tol, "compress")

    # a range that starts and ends inside a tile, with the partial sum of a ring added
    first, count = slices // 5 + 1, slices // 2 + 1
    part = torch.randn(slices * k, device=DEV)
    out = torch.full((slices * k,), 7.0, device=DEV)
    b.compress_segment(g, N, first, count, part, out)
    got = out.cpu().numpy().reshape(slices, k)
    assert np.all(got[:first] == 7.0) and np.all(got[first + count:] == 7.0)
    p = part.cpu().numpy().reshape(slices, k).astype(np.float64)
    _close(got[first:first + count], (want + p)[first:first + count], tol, "segment")

    yd = y.cpu().numpy().astype(np.float64).reshape(slices, k)
    back = np.einsum("sdk,sk->sd", U, yd) + mu
    for odt in ("f32", "bf16"):
        r = torch.full((M + 8,), 7.0, device=DEV, dtype=torch.bfloat16 if odt == "bf16" else torch.float32)
        b.decompress(y, r[:M], odt)
        got = r.to(torch.float64).cpu().numpy()
        assert np.all(got[M:] == 7.0)
        _close(got[:M], back.reshape(-1)[:M], 2.0 ** -8 if odt == "bf16" else tol, f"decompress to {odt}")
        r.fill_(7.0)
        b.decompress_segment(y, first, count, r[:M], odt)
        seg = r.to(torch.float64).cpu().numpy()
        lo, hi = first * d, min(M, (first + count) * d)
        assert np.array_equal(seg[lo:hi], got[lo:hi]) and np.all(seg[:lo] == 7.0) and np.all(seg[hi:] == 7.0)

    gvq.gvq_set_option(2, 1 if exact else 3)
    try:
        y2 = torch.empty_like(y)
        b.compress(g, N, y2)
        r2 = torch.empty(M, device=DEV)
        b.decompress(y, r2, "f32")
    finally:
        gvq.gvq_set_option(2, 0)
    r = torch.empty(M, device=DEV)
    b.decompress(y, r, "f32")
    _close(y.cpu().numpy(), y2.cpu().numpy(), tol, "compress, other route")
    _close(r.cpu().numpy(), r2.cpu().numpy(), tol, "decompress, other route")
    b.close()


@pytest.mark.parametrize("d,k", [(13, 3), (30, 7), (100, 25), (201, 50), (513, 128)])
def test_nan_and_infinity_stay_in_their_slice(d, k):
    rng = np.random.default_rng(d)
    slices = 300
    b, g, U, mu, x = _make(d, k, "f32", None, slices * d, rng)
    bad = {0: float("nan"), 63: float("inf"), 64: float("nan"), 150: float("-inf"), slices - 1: float("nan")}
    for s, v in bad.items():
        g[s * d + (s * 7) % d] = v
    y = torch.empty(slices * k, device=DEV)
    b.compress(g, 2, y)
    fine = np.isfinite(y.cpu().numpy().reshape(slices, k)).all(1)
    assert [int(s) for s in np.where(~fine)[0]] == sorted(bad)
    r = torch.empty(slices * d, device=DEV)
    b.decompress(y, r)
    if 2.0 * d * k / (4.0 * (d + k)) < 10.0:   # exact products: an infinity stays one, wherever in the slice it is
        g[63 * d:64 * d] = 1.0
        for e in range(d):
            g[63 * d + e] = float("inf")
            b.compress(g, 2, y)
            assert torch.isinf(y[63 * k:64 * k]).all(), e
            g[63 * d + e] = 1.0
        z = torch.zeros(slices * k, device=DEV)
        for c in range(k):
            z[63 * k + c] = float("inf")
            rz = torch.empty(slices * d, device=DEV)
            b.decompress(z, rz)
            assert torch.isinf(rz[63 * d:64 * d]).all(), c
            z[63 * k + c] = 0.0
    fine = np.isfinite(r.cpu().numpy().reshape(slices, d)).all(1)
    assert [int(s) for s in np.where(~fine)[0]] == sorted(bad)
    b.close()


def _einsum_close(got, want, tol, what):
    err = float((got.double() - want).abs().max() / want.abs().max())
    assert err <= tol, f"{what}: {err:.2e}"   # a NaN fails, too


def _uneven_cuts(S, B, rng):
    """B bases: most of them a few slices short or long, some of a single slice, some longer than any tile."""
    w = rng.choice([0.01, 1.0, 3.0, 40.0], B, p=[0.2, 0.5, 0.2, 0.1]) * rng.uniform(0.5, 1.5, B)
    cuts = np.concatenate([[0], 1 + np.arange(B) + np.floor(np.cumsum(w) / w.sum() * (S - B)).astype(np.int64)])
    cuts[-1] = S
    assert (np.diff(cuts) >= 1).all()
    return cuts


def _check_on_device(b, d, k, B, cuts, M, dtype, rng, N=3):
    """Eqs. (2) and (4), and a ring step over a range, against float64 on the device."""
    S = -(-M // d)
    U = torch.from_numpy(np.linalg.qr(rng.standard_normal((B, d, k)))[0].astype(np.float32))
    mu = torch.from_numpy((0.3 * rng.standard_normal((B, d))).astype(np.float32))
    b.import_(U.numpy(), mu.numpy())
    gen = torch.Generator(device=DEV).manual_seed(int(rng.integers(1 << 30)))
    g = torch.randn(M, device=DEV, generator=gen).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    x = torch.zeros(S * d, device=DEV, dtype=torch.float64)
    x[:M] = g.double()
    x = x.view(S, d)
    U, mu = U.to(DEV).double(), mu.to(DEV).double()
    want = torch.empty(S, k, device=DEV, dtype=torch.float64)
    for i in range(B):
        lo, hi = int(cuts[i]), int(cuts[i + 1])
        want[lo:hi] = (x[lo:hi] - mu[i] / N) @ U[i]
    tol = 2e-6 if 2.0 * d * k / (4.0 * (d + k)) < 10.0 else 4e-5
    y = torch.full((S * k,), float("nan"), device=DEV)
    b.compress(g, N, y)
    _einsum_close(y.view(S, k), want, tol, "compress")

    first, count = S // 7 + 5, S // 2 + 3
    part = torch.randn(S * k, device=DEV, generator=gen)
    out = torch.full((S * k,), 7.0, device=DEV)
    b.compress_segment(g, N, first, count, part, out)
    o = out.view(S, k)
    assert (o[:first] == 7.0).all() and (o[first + count:] == 7.0).all()
    _einsum_close(o[first:first + count], (want + part.view(S, k).double())[first:first + count], tol, "ring step")

    back = torch.empty(S, d, device=DEV, dtype=torch.float64)
    yd = y.view(S, k).double()
    for i in range(B):
        lo, hi = int(cuts[i]), int(cuts[i + 1])
        back[lo:hi] = yd[lo:hi] @ U[i].T + mu[i]
    for odt in ("f32", "bf16"):
        r = torch.full((M + 8,), 7.0, device=DEV, dtype=torch.bfloat16 if odt == "bf16" else torch.float32)
        b.decompress(y, r[:M], odt)
        assert (r[M:] == 7.0).all()
        _einsum_close(r[:M], back.view(-1)[:M], 2.0 ** -8 if odt == "bf16" else tol, f"decompress to {odt}")
        seg = torch.full_like(r, 7.0)
        b.decompress_segment(y, first, count, seg[:M], odt)
        lo, hi = first * d, min(M, (first + count) * d)
        assert torch.equal(seg[lo:hi], r[lo:hi]) and (seg[:lo] == 7.0).all() and (seg[hi:] == 7.0).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,k", [(24, 6), (40, 10), (100, 25), (201, 50)])
def test_many_short_bases(d, k, dtype):
    """Thousands of bases of a few dozen slices: right, and not slower than the kernels that search for a tile's basis (whose
    time per tile does not depend on the number of bases; measured at about their time or below, the bound leaves 2x)."""
    rng = np.random.default_rng(d)
    B = 3000 if d < 200 else 1500
    S = 37 * B
    cuts = np.arange(B + 1) * 37
    M = S * d - d // 3
    b = gvq.Basis(M, d, k, cuts, dtype)
    _check_on_device(b, d, k, B, cuts, M, dtype, rng)

    g = torch.randn(M, device=DEV).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    y, r = torch.randn(S * k, device=DEV), torch.empty_like(g)

    def best_of(f):
        f()
        times = []
        for _ in range(5):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(5):
                f()
            t1.record()
            torch.cuda.synchronize()
            times.append(t0.elapsed_time(t1))
        return min(times)

    exact = 2.0 * d * k / (4.0 * (d + k)) < 10.0
    for what, f in (("compress", lambda: b.compress(g, 3, y)), ("decompress", lambda: b.decompress(y, r))):
        here = best_of(f)
        gvq.gvq_set_option(2, 1 if exact else 3)
        try:
            there = best_of(f)
        finally:
            gvq.gvq_set_option(2, 0)
        assert here <= 2.0 * there, f"{what}: {here / 5:.3f} ms, LDS-tiled kernels {there / 5:.3f} ms"
    b.close()


# a shape for every compiled instance of the two kernels (the list is checked against the plans in test_flow_plan.py)
INSTANCES = [(9, 1), (25, 17), (41, 1), (41, 33), (41, 41), (49, 33), (57, 17), (57, 31), (57, 49), (73, 1), (73, 29), (73, 33),
             (89, 17), (89, 26), (89, 49), (105, 1), (105, 25), (105, 33), (105, 97), (121, 17), (137, 1), (137, 25), (137, 65),
             (137, 97), (169, 1), (169, 23), (169, 65), (201, 1), (201, 23), (201, 65), (233, 1), (233, 22), (233, 33), (265, 1),
             (265, 22), (265, 97), (329, 1), (329, 22), (329, 65), (393, 1), (393, 22), (393, 65), (393, 97), (521, 33), (521, 65),
             (521, 97), (649, 33), (649, 65), (777, 1), (777, 21), (777, 33), (777, 65), (905, 1), (905, 21), (905, 33)]
INSTANCE_ELEMENTS = 24_000_000   # at least three tiles for every work-group


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("blocks", [1, 60])
@pytest.mark.parametrize("d,k", INSTANCES)
def test_every_instance_with_several_tiles_per_work_group(d, k, blocks, dtype):
    """The steady loop of the kernels: the next tile asked for under this one, the last one's results leaving under it, changes of
    basis inside a work-group (bases shorter and longer than a tile, of one slice, ending anywhere), a ragged end, a range that
    starts and ends inside a tile; then other schedules (one work-group per compute unit, runs of one and of three tiles), which
    must not change a bit."""
    rng = np.random.default_rng(100 * d + k)
    M = INSTANCE_ELEMENTS - INSTANCE_ELEMENTS % d + d // 2 + 1
    S = -(-M // d)
    cuts = np.array([0, S]) if blocks == 1 else _uneven_cuts(S, blocks, rng)
    b = gvq.Basis(M, d, k, None if blocks == 1 else cuts, dtype)
    _check_on_device(b, d, k, blocks, cuts, M, dtype, rng)

    g = torch.randn(M, device=DEV).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    y, r = torch.empty(S * k, device=DEV), torch.empty_like(g)
    b.compress(g, 3, y)
    b.decompress(y, r)
    try:
        for wg_per_cu, run in ((1, 0), (0, 1), (1, 3)):
            gvq.gvq_set_option(0, wg_per_cu)
            gvq.gvq_set_option(1, run)
            y2, r2 = torch.full_like(y, float("nan")), torch.full_like(r, float("nan"))
            b.compress(g, 3, y2)
            b.decompress(y, r2)
            assert torch.equal(y, y2) and torch.equal(r, r2), (wg_per_cu, run)
    finally:
        gvq.gvq_set_option(0, 0)
        gvq.gvq_set_option(1, 0)
    b.close()


@pytest.mark.parametrize("d,k,dtype,S,bases,here", [
    (16, 1, "f32", 1_000_000, 1, True), (16, 5, "f32", 1_000_003, 3200, True), (16, 5, "f32", 1_000_003, 3300, False),
    (16, 15, "bf16", 1_000_000, 7, True), (16, 2, "bf16", 500_000, 1, True), (16, 2, "bf16", 490_000, 1, False),
    (32, 3, "bf16", 200_001, 1, True), (32, 3, "bf16", 480_000, 7, False), (32, 3, "bf16", 500_001, 3300, False),
    (32, 30, "f32", 1_000_001, 1, True), (32, 30, "f32", 1_000_001, 12_900, True), (32, 31, "bf16", 200_001, 7, True),
    (32, 31, "bf16", 190_001, 1, False), (64, 19, "f32", 500_000, 1, True), (64, 29, "f32", 500_009, 7, True),
    (64, 29, "bf16", 500_009, 2600, True), (64, 25, "bf16", 500_009, 1, True), (64, 23, "bf16", 500_009, 1, False),
    (64, 17, "f32", 500_009, 7, False), (64, 31, "bf16", 500_009, 1, False)])
def test_short_slices_with_ragged_comps(d, k, dtype, S, bases, here):
    """Compress of many slices of 16, 32 or 64 elements whose comps are no whole words, on both sides of the rule that sends them
    to these kernels or to the register-resident ones: whole gradients with a ragged tail, segments, the fused ring step,
    against float64.  d exact products added in fp32 are within d 2^-24 sum |u x| of the exact sum, and sum |u x| <= |x| for a unit
    column; the mean divided by N and what is left of it taken from x: two roundings more of |x| + |mu| / N.  Which kernels were
    taken shows in the last bits: option 2 leaves these kernels out."""
    gen = torch.Generator(device=DEV).manual_seed(d * k)
    M = S * d - (d // 2 + 1)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = (torch.randn(M, generator=gen, device=DEV) + 0.5).to(tdt)
    offs = [S * i // bases for i in range(bases + 1)]
    b = gvq.Basis(M, d, k, offs if bases > 1 else None, dtype)
    rng = np.random.default_rng(k)
    U = np.linalg.qr(rng.standard_normal((bases, d, k)))[0].astype(np.float32)
    mu = rng.standard_normal((bases, d)).astype(np.float32)
    b.import_(U, mu)
    U, mu = torch.from_numpy(U).to(DEV).double(), torch.from_numpy(mu).to(DEV).double()
    whole = torch.zeros(S * d, device=DEV, dtype=torch.float64)
    whole[:M] = x.double()
    whole = whole.view(S, d)
    want, tol = torch.empty(S, k, device=DEV, dtype=torch.float64), whole.norm(dim=1, keepdim=True)
    for i in range(bases):
        rows = slice(offs[i], offs[i + 1])
        want[rows] = (whole[rows] - mu[i] / 3) @ U[i]
        tol[rows] += mu[i].norm() / 3
    tol *= (d + 2) * 2.0 ** -24
    first, count = S // 3 + 1, S // 2 + 5
    part = torch.randn(S * k, generator=gen, device=DEV)
    got = []
    for mode in (0, 3):
        y, z = torch.full((S * k,), 7.0, device=DEV), torch.full((S * k,), 7.0, device=DEV)
        try:
            gvq.gvq_set_option(2, mode)
            b.compress(x, 3, y)
            b.compress_segment(x, 3, first, count, part, z)
        finally:
            gvq.gvq_set_option(2, 0)
        got.append((y.view(S, k), z.view(S, k)))
    rows = slice(first, first + count)
    outside = torch.ones(S, dtype=torch.bool, device=DEV)
    outside[rows] = False
    for y, z in got:
        assert bool(((y.double() - want).abs() <= tol).all())
        assert torch.equal(z[rows], y[rows] + part.view(S, k)[rows])
        assert bool((z[outside] == 7.0).all())
    if not here or bases > 1 or (dtype == "bf16" and d > 16):   # otherwise both add in the same order
        assert torch.equal(got[0][0], got[1][0]) != here
    b.close()
