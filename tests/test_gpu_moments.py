"""Covariance and sample count of the basis refresh at the edges of its tiles: slice lengths around the multiples of 16 and
128 at which the number of tiles or panels changes, lengths whose slices start off the word grid, lengths below one word,
chunks that end inside a block of samples, several bases, more gradients than one launch takes."""
import numpy as np
import pytest

from paper_1811_03617_amd import gvq

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [2, 3, 4, 5, 15, 16, 17, 30, 33, 47, 63, 64, 66, 79, 81, 96, 97, 100, 111, 113, 127, 128, 129,
                               160, 193, 255, 257, 383, 385, 513, 641, 897, 1023, 1024])
def test_covariance_and_counts(d, dtype):
    rng = np.random.default_rng(d)
    slices = 700 if d <= 128 else 260
    cuts = [0, slices // 3 + 1, slices // 3 + 2, slices] if d <= 300 else None   # a basis of one slice among them
    M = slices * d - (1 if d % 3 else 0)                                         # a ragged or a whole last slice
    L = 34 if d in (5, 128) else 3
    grads = [torch.from_numpy((rng.standard_normal(M) * rng.uniform(0.1, 2.0) + 0.3).astype(np.float32)) for _ in range(L)]
    if dtype == "bf16":
        grads = [g.to(torch.bfloat16) for g in grads]
    b = gvq.Basis(M, d, 1, cuts, dtype)
    b.fit([g.to(DEV) for g in grads])
    C, n = b.export_cov()
    mu = b.export()[1]
    b.close()
    X = np.stack([g.to(torch.float64).numpy()[: M // d * d].reshape(-1, d) for g in grads])
    for i, (lo, hi) in enumerate(zip(*((cuts or [0, slices])[k:] for k in (0, 1)))):
        x = X[:, lo:min(hi, M // d)].reshape(-1, d)
        assert n[i] == x.shape[0]
        if not len(x):
            continue
        m = x.mean(0)
        # n products summed in any order, then divided: at most n + 2 roundings of a sum of |products| (here n <= 23800)
        bound = (n[i] + 4) * 2.0 ** -53 * (np.abs(x).T @ np.abs(x) / n[i] + 2 * np.outer(np.abs(m), np.abs(m)))
        assert np.all(np.abs(C[i] - (x.T @ x / n[i] - np.outer(m, m))) <= 2 * bound + 1e-300)
        assert np.array_equal(C[i], C[i].T)
        assert np.allclose(mu[i], m, rtol=1e-6, atol=1e-7)
