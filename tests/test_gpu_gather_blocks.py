"""Where a gather of many blocks puts them: products with the identity on one
leg return every block of the other factor, permuted and bit for bit (sums of
one value and zeros), block by block, with few pieces and with more than a
thousand."""
import numpy as np
import pytest

import paper_1808_10804_amd as st

pytestmark = pytest.mark.gpu

SMALL = ({-1: 5, 0: 12, 1: 6, 2: 1}, {-1: 3, 0: 7, 1: 2}, {-1: 2, 0: 4, 1: 1})
LARGE = ({-1: 37, 0: 150, 1: 41, 2: 1}, {-1: 3, 0: 18, 1: 5}, {-1: 6, 0: 9, 1: 2})


@pytest.mark.parametrize("perm", [None, (0, 1, 3, 2), (2, 0, 3, 1), (3, 2, 1, 0)])
@pytest.mark.parametrize("leg", [0, 2])
@pytest.mark.parametrize("sizes", [SMALL, LARGE], ids=["few", "many"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_every_block_in_its_place(dtype, sizes, leg, perm):
    q, x, y = sizes
    A = st.Tensor.create([(q, 1), (x, 1), (q, -1), (y, -1)], 0, dtype)
    A.upload(np.random.default_rng(leg).standard_normal(A.nnz))
    eye = st.Tensor.create([(q, 1), (q, -1)], 0, dtype)
    eye.upload(np.concatenate([np.eye(shape[0]).reshape(-1) for _, shape, _, _ in eye.blocks()]))
    out = st.contract(A, eye, [leg], [0 if leg == 2 else 1], out_perm=perm, prec=dtype)
    order = [l for l in range(4) if l != leg] + [leg]   # free legs of A, then the identity's
    order = [order[p] for p in (perm or range(4))]
    want = A.block_dict()
    got = out.block_dict()
    assert len(got) == len(want)
    for label, block in want.items():
        at = tuple(label[l] for l in order)
        assert np.array_equal(got[at], block.transpose(order)), (label, block.shape)
