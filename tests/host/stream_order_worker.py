"""One scenario of test_stream_order_host.py, run with the HIP runtime without a
GPU (fake_hip.cpp) preloaded; exits with 0 if it holds."""
import ctypes as C
import sys
import threading

sys.modules["torch"] = None   # its import would bring a HIP runtime of its own
import numpy as np            # noqa: E402

import paper_1808_10804_amd as st   # noqa: E402

fake = C.CDLL(None)
fake.fake_stream.restype = C.c_void_p
S = fake.fake_stream()


def su2(legs, seed):
    t = st.Tensor.create(legs, dtype="f64", group="su2")
    return t.upload(np.random.default_rng(seed).standard_normal(t.nnz))


def su2_double_layer():
    """The fusion matrices of an SU(2) double layer go into blocks that
    another stream released and whose work is still queued there."""
    v = {0: 1, 1: 2}
    A = su2([({1: 1}, 1), (v, 1), (v, 1), (v, -1), (v, -1)], 1)
    B, D = su2([(v, 1), (v, -1)], 2), su2([(v, 1), (v, -1)], 3)
    other = fake.fake_stream()
    for _ in range(20):
        st.contract(B, D, [1], [0], prec="f64", stream=other)
    st.double_layer(A, stream=S)


def su2_move():
    """The fusion isometries of an SU(2) move, kept for later moves, are built
    while the corners are still queued (kernels do nothing here, so the move
    ends at its cut)."""
    for chi in ({0: 3, 1: 4, 2: 2}, {0: 4, 1: 3, 2: 2}):
        dd = {0: 2, 1: 3, 2: 2}
        C4 = [su2([(chi, 1), (chi, -1)], i) for i in range(4)]
        T4 = [su2([(chi, 1), (dd, -1 if i in (0, 3) else 1), (chi, -1)], i + 4) for i in range(4)]
        a = su2([(dd, 1), (dd, 1), (dd, -1), (dd, -1)], 9)
        env = st.CtmEnv(C4, T4)
        try:
            env.move(a, 12, prec="f64", stream=S)
        except st.SymtenError as e:
            print(e)


def _matrices(n, seed):
    ts = [st.Tensor.create([({0: n}, 1), ({0: n}, -1)], 0, "f64") for _ in range(2)]
    return [t.upload(np.random.default_rng(seed + i).standard_normal(n * n)) for i, t in enumerate(ts)]


def new_plan_beside_another_thread():
    """While a contraction seen for the first time waits for its stream before
    it writes its tables, one of another thread and stream goes through."""
    A, B = _matrices(20, 1)
    X, Y = _matrices(21, 3)
    other = fake.fake_stream()
    for _ in range(3):
        st.contract(X, Y, [1], [0], prec="f64", stream=other)
        st.contract(X, Y, [1], [0], prec="f64", stream=S)   # leaves used blocks to S
    through = []

    def elsewhere():
        st.contract(X, Y, [1], [0], prec="f64", stream=other)
        st.sync(other)

    @C.CFUNCTYPE(None)
    def meanwhile():
        t = threading.Thread(target=elsewhere, daemon=True)
        t.start()
        t.join(5)
        through.append(not t.is_alive())

    fake.fake_during_sync(meanwhile)
    st.contract(A, B, [1], [0], prec="f64", stream=S)
    assert through == [True], through


if __name__ == "__main__":
    scenario = globals().get(sys.argv[1])
    if scenario:
        scenario()
    else:
        check = getattr(fake, sys.argv[1])()   # those of fake_hip.cpp
        if check:
            sys.exit(f"{sys.argv[1]}: check {check} failed")
    n = fake.fake_hazards()
    if n:
        sys.exit(f"{sys.argv[1]}: {n} copies into memory that queued work may use")
