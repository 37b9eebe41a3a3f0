"""GPU tests of the FP64 kernels at the edges of the tile and of the k-step, on
padded and 8-byte aligned operands whose padding holds NaN, and of the double
complex ones on odd sizes.

Bar: element by element |C - AB| <= (k + 2) 2^-53 (|A||B|)_ij, against the same
product in long double (complex: (2 k + 4) 2^-53, each part a sum of 2k
products)."""
import numpy as np
import pytest

from paper_2305_01024_amd import ftgemm as F

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def handles():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hs = (F.ftgemm_create(F.F64, 0), F.ftgemm_create(F.C64, 0))
    yield hs
    for h in hs:
        F.ftgemm_destroy(h)


def _padded(X, ld, offset):
    import torch
    m, n = X.shape
    buf = np.full(offset + ld * n, np.nan, X.dtype)
    buf[offset:].reshape(n, ld)[:, :m] = X.T
    d = torch.from_numpy(buf).cuda()
    return d, d.data_ptr() + X.itemsize * offset


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 1, 2), (3, 5, 3), (5, 1, 17), (127, 130, 15), (129, 126, 16),
                                   (131, 257, 33), (254, 3, 47), (257, 255, 31), (256, 128, 64), (130, 129, 1)])
def test_edges(handles, shape):
    import torch
    m, n, k = shape
    r = np.random.default_rng(m * 5 + n * 3 + k)
    A, B = r.standard_normal((m, k)), r.standard_normal((k, n))
    ref = A.astype(np.longdouble) @ B.astype(np.longdouble)
    bound = (k + 2) * 2.0 ** -53 * (np.abs(A) @ np.abs(B))
    for level in (0, 1, 2):
        for pa, pb, offset in ((0, 0, 0), (1, 3, 1), (2, 1, 3)):
            dA, qA = _padded(A, m + pa, offset)
            dB, qB = _padded(B, k + pb, offset)
            dC = torch.zeros((n, m), device="cuda", dtype=torch.float64)
            rep = F.ReportBuffer(64)
            st = F.ftgemm_run_f64(handles[0], m, n, k, 1.0, qA, m + pa, qB, k + pb, 0.0, dC.data_ptr(), m, level, 0.0,
                                  torch.cuda.current_stream().cuda_stream, rep)
            assert st == F.OK and rep.report.n_events == 0
            assert np.all(np.abs(dC.cpu().numpy().T - ref) <= bound)


@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 7), (129, 67, 33), (130, 131, 40)])
def test_complex_odd_sizes(handles, shape):
    import torch
    m, n, k = shape
    r = np.random.default_rng(m + n + k)
    A = r.standard_normal((m, k)) + 1j * r.standard_normal((m, k))
    B = r.standard_normal((k, n)) + 1j * r.standard_normal((k, n))
    ref = A.astype(np.clongdouble) @ B.astype(np.clongdouble)
    bound = 2 * (2 * k + 4) * 2.0 ** -53 * (np.abs(A) @ np.abs(B))
    dA, qA = _padded(A, m + 1, 1)
    dB, qB = _padded(B, k + 2, 1)
    dC = torch.zeros((n, m), device="cuda", dtype=torch.complex128)
    rep = F.ReportBuffer(64)
    st = F.ftgemm_run_z64(handles[1], m, n, k, 1.0, qA, m + 1, qB, k + 2, 0.0, dC.data_ptr(), m, 2, 0.0,
                          torch.cuda.current_stream().cuda_stream, rep)
    assert st == F.OK and rep.report.n_events == 0
    assert np.all(np.abs(dC.cpu().numpy().T - ref) <= bound)
