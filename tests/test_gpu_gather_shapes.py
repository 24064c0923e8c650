"""Gathers whose copies take each route of the kernel: runs along an outer dim
(whole, ragged, of the source's unit-stride dim), no runs (one dim, dims too
short for runs), tiles through LDS, zero fills, one or several thousand pieces;
against the dense product of the same blocks.  Also split-K reductions with a
ragged last tile.

The gather moves values unchanged, so the tolerance is that of the product: K
terms of standard normal numbers, an FP64 (FP32) sum of K <= 4096 terms off by
less than K eps times the largest partial sum (below 8 sqrt(K)), relative to a
largest entry of about 4 sqrt(K): 2 K eps, 2e-12 and 1e-3 at the most; FP32
sums in blocks of 32 and pairs stay below 1e-5 of it, bf16x3 (2^-16 per factor)
below 1e-4."""
import numpy as np
import pytest

import paper_1808_10804_amd as st

pytestmark = pytest.mark.gpu

# (dims of A, dims of B, legs of A, legs of B, out_perm): one sector per leg
SHAPES = [
    ((7,), (7, 4), (0,), (0,), None),                     # single dims
    ((5, 3), (3, 2), (1,), (0,), None),                   # dims below a run
    ((64, 9), (9, 33), (1,), (0,), None),                 # B transposed, no tile (9 < 16)
    ((3, 130, 13), (13, 130, 5), (1, 2), (1, 0), None),   # ragged runs, order of the pair swapped
    ((16, 24, 30), (24, 17, 16), (1, 0), (0, 2), None),   # runs along the source's unit dim
    ((16, 24, 31), (24, 18, 16), (1, 0), (0, 2), (1, 0)),
    ((70, 33, 6), (70, 40), (0,), (0,), None),            # tiles
    ((257, 1030), (1030, 259), (1,), (0,), None),         # split K, ragged tiles
    ((40, 11, 40, 12), (12, 11, 50), (1, 3), (1, 0), None),
    ((6, 300, 7, 300), (300, 6, 5), (1, 0), (0, 1), None),
]


def _dense(t, dims, rng):
    x = rng.standard_normal(dims)
    t.upload(x.reshape(-1))
    return x


@pytest.mark.parametrize("prec,tol", [("f64", 2e-12), ("f32", 1e-5), ("bf16x3", 1e-4)])
@pytest.mark.parametrize("case", range(len(SHAPES)))
def test_one_block(case, prec, tol):
    da, db, la, lb, perm = SHAPES[case]
    dt = "f64" if prec == "f64" else "f32"
    rng = np.random.default_rng(case)
    A = st.Tensor.create([({0: d}, 1) for d in da], 0, dt)
    B = st.Tensor.create([({0: d}, -1) for d in db], 0, dt)
    x, y = _dense(A, da, rng), _dense(B, db, rng)
    if dt == "f32":
        x, y = x.astype(np.float32).astype(np.float64), y.astype(np.float32).astype(np.float64)
    want = np.tensordot(x, y, (la, lb))
    if perm is not None:
        want = want.transpose(perm)
    out = st.contract(A, B, list(la), list(lb), out_perm=perm, prec=prec)
    got = np.asarray(out.download()).reshape(want.shape)
    assert np.abs(got - want).max() <= tol * max(np.abs(want).max(), 1e-30)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_many_sectors_and_pieces(dtype):
    """Several sectors per leg (zero fills, blocks of one element) and enough
    pieces for whole-piece workgroups: a product with the identity returns the
    block values themselves, bit for bit (sums of one value and zeros)."""
    rng = np.random.default_rng(5)
    q = {-1: 37, 0: 150, 1: 41, 2: 1}
    A = st.Tensor.create([(q, 1), ({-1: 3, 0: 18, 1: 5}, 1), (q, -1), ({-1: 6, 0: 9, 1: 2}, -1)], 0, dtype)
    I = st.Tensor.create([(q, 1), (q, -1)], 0, dtype)
    x = rng.standard_normal(A.nnz)
    A.upload(x)
    I.upload(np.concatenate([np.eye(shape[0]).reshape(-1) for _, shape, _, _ in I.blocks()]))
    out = st.contract(A, I, [2], [0], out_perm=[0, 1, 3, 2], prec=dtype)
    assert np.array_equal(np.sort(np.asarray(out.download())), np.sort(np.asarray(A.download())))
