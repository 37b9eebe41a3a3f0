"""GPU tests of the FP32 kernels that run on three-way bf16 splits: edges of
tiles and panels, padded and misaligned operands whose padding holds NaN, and
operands the split cannot hold (tiny, huge, Inf, NaN), which take the FP32
matrix instructions.

Bar: element by element |C - AB| <= (k + 2) 2^-24 (|A||B|)_ij, the bar of the
other FP32 tests.  A value too small for the split has an absolute error of
2^-24 of itself in that bound, so a split that dropped its last bits fails."""
import numpy as np
import pytest

from paper_2305_01024_amd import ftgemm as F

pytestmark = pytest.mark.gpu
CONFIGS = [(256, 256, 32, 8), (128, 128, 32, 8)]


@pytest.fixture(scope="module")
def h():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    handle = F.ftgemm_create(F.F32, 0)
    yield handle
    F.ftgemm_destroy(handle)


def _padded(X, ld, offset):
    """X column-major with leading dimension ld, `offset` floats into a buffer whose padding is NaN."""
    import torch
    m, n = X.shape
    buf = np.full(offset + ld * n, np.nan, np.float32)
    view = buf[offset:].reshape(n, ld)
    view[:, :m] = X.T
    d = torch.from_numpy(buf).cuda()
    return d, d.data_ptr() + 4 * offset


def _run(h, A, B, level, pad=(0, 0, 0), offset=0, beta=0.0, C0=None):
    import torch
    m, k = A.shape
    n = B.shape[1]
    lda, ldb, ldc = m + pad[0], k + pad[1], m + pad[2]
    dA, pA = _padded(A, lda, offset)
    dB, pB = _padded(B, ldb, offset)
    dC, pC = _padded(np.zeros((m, n), np.float32) if C0 is None else C0, ldc, offset)
    rep = F.ReportBuffer(64)
    st = F.ftgemm_run(h, m, n, k, 1.0, pA, lda, pB, ldb, beta, pC, ldc, level, 0.0,
                      torch.cuda.current_stream().cuda_stream, rep)
    full = dC.cpu().numpy()[offset:].reshape(n, ldc)
    assert np.isnan(full[:, m:]).all()      # C's padding is untouched
    return st, full[:, :m].T.copy(), rep


def _ratio(C, A, B):
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    bound = (A.shape[1] + 2) * 2.0 ** -24 * (np.abs(A64) @ np.abs(B64)) + 2.0 ** -149
    return np.max(np.abs(C - A64 @ B64) / bound)


@pytest.mark.parametrize("cfg", CONFIGS)
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 2, 3), (4, 4, 4), (5, 1, 17), (127, 130, 15), (129, 126, 16),
                                   (131, 257, 33), (254, 3, 47), (257, 255, 31), (256, 128, 64), (385, 130, 1)])
def test_edges(h, cfg, shape):
    m, n, k = shape
    r = np.random.default_rng(m * 7 + n * 3 + k)
    A, B = r.standard_normal((m, k)).astype(np.float32), r.standard_normal((k, n)).astype(np.float32)
    F.ftgemm_set_config(h, cfg)
    try:
        for level in (0, 1, 2):
            for pad, offset in (((0, 0, 0), 0), ((1, 3, 2), 1)):
                st, C, rep = _run(h, A, B, level, pad, offset)
                assert st == F.OK and rep.report.n_events == 0
                assert _ratio(C, A, B) <= 1.0
        C0 = r.standard_normal((m, n)).astype(np.float32)
        st, C, rep = _run(h, A, B, 2, (1, 0, 3), 3, 1.0, C0)
        assert st == F.OK and np.max(np.abs(C - C0 - A.astype(np.float64) @ B) /
                                     ((k + 4) * 2.0 ** -24 * (np.abs(A) @ np.abs(B) + np.abs(C0)))) <= 1.0
    finally:
        F.ftgemm_set_config(h, None)


@pytest.mark.parametrize("cfg", CONFIGS)
@pytest.mark.parametrize("level", [0, 1, 2])
@pytest.mark.parametrize("small", [2.0 ** -112, 2.0 ** -122, 2.0 ** -135])
def test_tiny_elements(h, cfg, level, small):
    """Rows of ordinary size whose products are zero but for tiny elements."""
    m, n, k = 300, 140, 70
    r = np.random.default_rng(5)
    A, B = r.standard_normal((m, k)).astype(np.float32), r.standard_normal((k, n)).astype(np.float32)
    B[:35, :] = 0.0                     # A's ordinary half meets zeros
    A[:, 35:] *= np.float32(small)
    B[35:, :] *= np.float32(2.0 ** 60)
    F.ftgemm_set_config(h, cfg)
    try:
        st, C, rep = _run(h, A, B, level)
    finally:
        F.ftgemm_set_config(h, None)
    assert st == F.OK and rep.report.n_events == 0
    assert _ratio(C, A, B) <= 1.0


@pytest.mark.parametrize("cfg", CONFIGS)
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_not_splittable(h, cfg, value):
    """One element that the split cannot hold: the tile is what FP32 arithmetic gives, the others are untouched."""
    m, n, k = 300, 270, 50
    r = np.random.default_rng(6)
    A, B = r.standard_normal((m, k)).astype(np.float32), r.standard_normal((k, n)).astype(np.float32)
    A[280, 20] = value
    B[20, 200] = 0.0 if np.isfinite(value) else B[20, 200]
    with np.errstate(all="ignore"):
        ref = (A.astype(np.float64) @ B.astype(np.float64)).astype(np.float32)
    F.ftgemm_set_config(h, cfg)
    try:
        for level in (0, 2):
            st, C, rep = _run(h, A, B, level)
            assert st in (F.OK, F.NONFINITE_INPUT)
            assert (level == 0) or (st == F.NONFINITE_INPUT and rep.report.nonfinite_input > 0)
            rows = np.arange(m) != 280
            assert _ratio(C[rows], A[rows], B) <= 1.0
            fine = np.abs(ref[280]) < 1e38
            assert np.array_equal(np.isnan(C[280]), np.isnan(ref[280]))
            assert np.array_equal(np.isinf(C[280])[~fine], np.isinf(ref[280])[~fine])
    finally:
        F.ftgemm_set_config(h, None)


@pytest.mark.parametrize("cfg", CONFIGS)
@pytest.mark.parametrize("value", [0.0, 1e-38])
def test_faults_beside_tiles_without(h, cfg, value):
    """Faults in the first and the last tile, each applied and corrected once,
    with every tile on the split (0) or some elements too small for it."""
    m = n = 300
    k = 512
    r = np.random.default_rng(21)
    A, B = r.standard_normal((m, k)).astype(np.float32), r.standard_normal((k, n)).astype(np.float32)
    if value:
        A[280, 20] = value      # the last row of tiles
        B[30, 5] = value        # the first column of tiles
    last = (m - 1) // cfg[0]
    sites = np.zeros(2, F.FAULT_DTYPE)
    sites["tile_m"] = sites["tile_n"] = (0, last)
    sites["kstep"], sites["row"], sites["col"] = (1, 9), (17, 30), (40, 20)
    sites["kind"], sites["payload"] = F.FAULT_ADD, 1e6
    F.ftgemm_set_config(h, cfg)
    F.ftgemm_set_injection(h, sites)
    try:
        st, C, rep = _run(h, A, B, 2)
        log = F.ftgemm_get_injection_log(h)
    finally:
        F.ftgemm_set_injection(h, None)
        F.ftgemm_set_config(h, None)
    assert st == F.OK and len(log) == 2 and rep.report.corrected == 2 and rep.report.n_events == 2
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    bound = (k + 2) * 2.0 ** -24 * (np.abs(A64) @ np.abs(B64))
    for t, row, col in ((0, 17, 40), (last, 30, 20)):
        i = t * cfg[0] + row
        bound[i, t * cfg[0] + col] += bound[i].sum()     # rebuilt from the row's checksum
    assert np.max(np.abs(C - A64 @ B64) / bound) <= 1.0


def test_tiles_of_a_batch(h):
    """The batch's FP32 tiles over ragged sizes against the products."""
    import torch
    r = np.random.default_rng(8)
    sizes = [(33, 47, 61), (128, 128, 128), (129, 250, 35), (255, 131, 300), (1, 300, 17), (70, 64, 64)]
    probs, keep = F.make_problems(len(sizes)), []
    for q, (m, n, k) in enumerate(sizes):
        A, B = r.standard_normal((m, k)).astype(np.float32), r.standard_normal((k, n)).astype(np.float32)
        dA, pA = _padded(A, m + 1, 1)
        dB, pB = _padded(B, k + 3, 1)
        dC, pC = _padded(np.zeros((m, n), np.float32), m, 0)
        probs[q] = (F.F32, 0, m, n, k, m + 1, k + 3, m, 1.0, 0.0, 1.0, 1.0, pA, pB, pC)
        keep.append((A, B, dA, dB, dC))
    rep = F.ReportBuffer(64)
    st = F.ftgemm_batched(h, probs, F.FT_CORRECT, 0.0, torch.cuda.current_stream().cuda_stream, rep)
    assert st == F.OK and rep.report.n_events == 0
    for (m, n, k), (A, B, dA, dB, dC) in zip(sizes, keep):
        assert _ratio(dC.cpu().numpy().reshape(n, m).T, A, B) <= 1.0
