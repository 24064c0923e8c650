"""The eigensolver of the projector stage at the edges of its register
shapes: a matrix is held by workgroups whose row and column slots are fixed
per range of orders, so the first and last order of every range, and jobs that
have to share or cross an XCD, take paths of their own.

Eigenvalues against LAPACK, and the residual and orthogonality of the vectors,
relative to max |lambda|: a Householder reduction and the steps after it leave
an error of a modest multiple of sqrt(n) ulps, 1e-13 for the orders here."""
import numpy as np
import pytest
import torch

import paper_1808_10804_amd as st

pytestmark = pytest.mark.gpu

TOL = 1e-13


def _check(sizes, k, seed):
    rng = np.random.default_rng(seed)
    mats = []
    for n in sizes:
        y = rng.standard_normal((n, n))
        mats.append(y + y.T)
    dev = [torch.from_numpy(m).to("cuda") for m in mats]
    out = st.eigh(dev, [min(k, n) for n in sizes])
    for n, m, (w, Z) in zip(sizes, mats, out):
        print(f"n = {n}", flush=True)
        w, Z = w.cpu().numpy(), Z.cpu().numpy()
        ref = np.linalg.eigvalsh(m)
        scale = np.max(np.abs(ref))
        assert np.max(np.abs(w - ref)) <= TOL * scale
        lam = w[::-1][:Z.shape[1]]
        assert np.max(np.linalg.norm(m @ Z - Z * lam, axis=0)) <= TOL * scale
        assert np.max(np.abs(Z.T @ Z - np.eye(Z.shape[1]))) <= TOL


@pytest.mark.parametrize("sizes", [
    [127, 128, 129, 191, 192, 193], [255, 256, 257, 383, 384, 385], [511, 512, 513, 703, 704, 705],
    [1023, 1024, 1025], [1536, 1537], [2048], [2049], [3073]])
def test_edges_of_the_register_shapes(sizes):
    _check(sizes, 5, 31 + sizes[0])


def test_jobs_spread_over_xcds_and_launches():
    """Twelve jobs of twenty workgroups: eight fill one XCD each, the others
    get workgroups of several; thirteen more jobs take a second launch."""
    _check([400] * 12, 3, 5)
    _check([400] * 13 + [90], 2, 6)


@pytest.mark.parametrize("sizes", [
    [705, 704, 385, 384, 383, 65, 1], [1025, 257, 256, 192, 2], [1537, 703, 511, 64]])
def test_jobs_of_all_sizes_in_one_launch(sizes):
    """Orders of the 256-thread variants beside larger ones, all held by 512."""
    _check(sizes, 4, 77 + sizes[0])
