"""The library's block pool hands a block released on one stream to calls on
another: results of contractions alternating between streams, whose panels and
outputs go round through the pool while earlier work is still queued, equal
those of one stream bit for bit; the same from two threads with a stream each."""
import threading

import numpy as np
import pytest
import torch

import paper_1808_10804_amd as st

pytestmark = pytest.mark.gpu

CHI = {-2: 40, 0: 60, 2: 40}
DD = {-2: 9, 0: 18, 2: 9}


def _operands(seed):
    rng = np.random.default_rng(seed)
    C = st.Tensor.create([(CHI, 1), (CHI, -1)], 0, "f32")
    T = st.Tensor.create([(CHI, 1), (DD, -1), (CHI, -1)], 0, "f32")
    for t in (C, T):
        t.upload(rng.standard_normal(t.nnz))
    torch.cuda.synchronize()
    return C, T


def _chain(C, T, stream):
    """C T, then T C of the result: several panels and intermediates released
    while the GPU still works on them."""
    X = st.contract(C, T, [1], [0], prec="f32", stream=stream)
    for _ in range(3):
        X = st.contract(X, C, [2], [0], prec="f32", stream=stream)
    return X


def test_alternating_streams():
    streams = [torch.cuda.Stream() for _ in range(3)]
    ops = [_operands(s) for s in range(3)]
    want = []
    for C, T in ops:
        want.append(_chain(C, T, 0).download())
    got = []
    for rep in range(20):
        for i, s in enumerate(streams):
            X = _chain(*ops[i], s.cuda_stream)
            got.append((i, X, s))
            if len(got) > 4:       # the oldest result is read and released
                j, Y, t = got.pop(0)
                t.synchronize()
                assert np.array_equal(Y.download(t.cuda_stream), want[j])
    torch.cuda.synchronize()
    for j, Y, t in got:
        assert np.array_equal(Y.download(t.cuda_stream), want[j])


def test_threads_with_a_stream_each():
    ops = [_operands(10 + s) for s in range(4)]
    want = [_chain(C, T, 0).download() for C, T in ops]
    torch.cuda.synchronize()
    bad = []

    def work(i):
        s = torch.cuda.Stream()
        for _ in range(15):
            X = _chain(*ops[i], s.cuda_stream)
            s.synchronize()
            if not np.array_equal(X.download(s.cuda_stream), want[i]):
                bad.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert bad == []
