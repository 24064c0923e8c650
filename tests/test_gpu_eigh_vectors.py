"""The eigensolver on matrices that the random ones of the other tests do not
resemble; eigenvalues, residuals and orthogonality with the bound of those
tests, 1e-13 relative to max |lambda|."""
import numpy as np
import pytest
import torch

import paper_1808_10804_amd as st

pytestmark = pytest.mark.gpu

TOL = 1e-13


def _solve(m, k):
    w, Z = (x.cpu().numpy() for x in st.eigh([torch.from_numpy(m).to("cuda")], [k])[0])
    ref = np.linalg.eigvalsh(m)
    scale = np.max(np.abs(ref))
    assert np.max(np.abs(w - ref)) <= TOL * scale
    assert np.all(np.isfinite(Z))
    return w, Z, scale


@pytest.mark.parametrize("weakest", [20, 30, 40, 60])
def test_couplings_below_rounding(weakest):
    """Tridiagonal matrices of small integers whose parts are coupled by numbers
    far below rounding: the ratios of neighbouring entries of a vector reach
    1e+-200, and their products over parts of it leave the range of FP64 where
    the entries do not."""
    for seed in range(60):
        rng = np.random.default_rng(seed)
        n = int(rng.integers(40, 120)) * 2 + 1
        d = np.round(rng.standard_normal(n))
        e = np.ones(n - 1)
        weak = rng.random(n - 1) < 0.5
        e[weak] = 10.0 ** -rng.uniform(weakest / 2, weakest, int(weak.sum()))
        print(f"seed = {seed}, n = {n}", flush=True)
        _solve(np.diag(d) + np.diag(e, 1) + np.diag(e, -1), n)


@pytest.mark.parametrize("n", [1, 2, 65, 129, 400, 800])
@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("where", ["corner", "inside", "all"])
def test_not_finite(n, value, where):
    """No eigenvalue comes out of a matrix with NaN or Inf in it as a number;
    matrices solved beside it are not touched by it."""
    rng = np.random.default_rng(n)
    m = rng.standard_normal((n, n))
    m = m + m.T
    good = m.copy()
    i, j = {"corner": (0, 0), "inside": (n // 2, n // 3), "all": (slice(None), slice(None))}[where]
    m[i, j] = m[j, i] = value
    print(f"n = {n}", flush=True)
    (w, _), (v, Z) = st.eigh([torch.from_numpy(x).to("cuda") for x in (m, good)], [0, 1])
    assert not np.any(np.isfinite(w.cpu().numpy()))
    ref = np.linalg.eigvalsh(good)
    assert np.max(np.abs(v.cpu().numpy() - ref)) <= TOL * np.max(np.abs(ref))
    assert np.all(np.isfinite(Z.cpu().numpy()))


@pytest.mark.parametrize("n", [200, 700, 1100])
@pytest.mark.parametrize("count,gap", [(10, 1.05e-3), (40, 1.1e-3)])
def test_values_beside_a_multiplet(n, count, gap):
    """Multiplets of `count` equal eigenvalues, each with single ones `gap`
    ||T|| away on both sides, just beyond where close values are taken for a
    cluster: their vectors are orthogonal to every member of the multiplet."""
    for seed in range(6):
        rng = np.random.default_rng(n + count + 1000 * seed)
        q, _ = np.linalg.qr(rng.standard_normal((n, n)))
        top = []
        for g in range(3):
            c = 1.0 - 4 * gap * g
            top += [c] + [c - gap] * count + [c - 2 * gap]
        m = (q * np.concatenate([top, 0.5 * rng.random(n - len(top))])) @ q.T
        m = 0.5 * (m + m.T)
        k = len(top)
        print(f"n = {n}, seed = {seed}", flush=True)
        w, Z, scale = _solve(m, k)
        assert np.max(np.linalg.norm(m @ Z - Z * w[::-1][:k], axis=0)) <= TOL * scale
        assert np.max(np.abs(Z.T @ Z - np.eye(k))) <= TOL
