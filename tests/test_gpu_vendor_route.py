"""Moves with a sector that the library's own eigensolver does not hold (orders
above 3328, in FP64 a side above 2048): they go to rocSOLVER, with the Gram
matrix in FP32 and the Jordan-Wielandt matrix in FP64.  One bond of the right
edge is wide and all others are small, so the oracle stays cheap.  Kept
singular values and the left column against the dense oracle, with the
tolerances of the moves: 1e-12 in FP64, 1e-5 in FP32."""
import numpy as np
import pytest

import paper_1808_10804_amd as st
from oracle import ctm, u1
from workload import from_dense, to_dense, rel

pytestmark = pytest.mark.gpu

DD, CHI = {0: 16}, 8


def _draw(rng, legs, dtype):
    x = rng.standard_normal([sum(s.values()) for s, _ in legs])
    return x.astype(np.float32).astype(np.float64) if dtype == "f32" else x


@pytest.mark.parametrize("prec,tol", [("f64", 1e-12), ("f32", 1e-5)])
@pytest.mark.parametrize("wide,own", [(40, True), (209, False)])
def test_wide_sector(prec, tol, wide, own):
    bonds = [{0: 4}] * 8
    bonds[3] = {0: wide}   # T2-C3: the upper half reaches 16 `wide` right-hand states
    rng = np.random.default_rng(wide)
    C, T, Cd, Td = [], [], [], []
    for i in range(4):
        legs = [(bonds[2 * i - 1], 1), (bonds[2 * i], -1)]
        C.append(_draw(rng, legs, prec))
        Cd.append(from_dense(C[-1], legs, dtype=prec))
        legs = [(bonds[2 * i], 1), (DD, -1 if i in (0, 3) else 1), (bonds[2 * i + 1], -1)]
        T.append(_draw(rng, legs, prec))
        Td.append(from_dense(T[-1], legs, dtype=prec))
    legs = [(DD, 1), (DD, 1), (DD, -1), (DD, -1)]
    a = _draw(rng, legs, prec)
    env, ad = st.CtmEnv(Cd, Td), from_dense(a, legs, dtype=prec)
    print(f"wide = {wide}, {prec}", flush=True)
    st.profile_begin()
    env.move(ad, CHI, prec=prec)
    assert any(k["name"].startswith("eigh_") for k in st.profile_end()) == own
    C1, T4, C4, s = ctm.left_move(C, T, a, CHI)
    sv = np.sort(env.singular_values())[::-1]
    assert np.max(np.abs(sv[:len(s)] - s)) <= tol * s[0]
    k1, k4, kt = (to_dense(env.get(i)) for i in (0, 3, 7))
    assert rel(u1.left_column(k1, kt, k4), u1.left_column(C1, T4, C4)) <= tol
