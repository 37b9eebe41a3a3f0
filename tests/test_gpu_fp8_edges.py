"""GPU tests of the FP8 kernels at the edges of tiles and panels, on padded and
misaligned operands whose padding holds NaN, and with a fault in every block
of a tile.

Bar: element by element |C - AB| <= ceil(k / 64) 2^-14 (|A||B|)_ij on the
decoded operands: the instruction sums its 64 products as if rounded to about
16 bits (2.6e-5 of (|A||B|)_ij measured over one instruction), with a factor of
two above that.  (Products of a few rows and k are left out where that rounding
alone exceeds the FP32 threshold of the checks, which for FP8 is empirical:
4 x 4 x 8 logs an event with any of the library's FP8 kernels.)"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2305_01024_amd import ftgemm as F
from paper_2305_01024_amd import workloads as W

from gpu_util import event_keys, replay_against_gpu

pytestmark = pytest.mark.gpu
CONFIGS = [(256, 256, 64, 4), (128, 128, 64, 4)]
KINDS = {"fp8": (F.F8E4M3, W.quantize_e4m3, O.decode_e4m3, np.uint8, 0x7f)}


def _u(k):
    return -(-k // 64) * 2.0 ** -14



@pytest.fixture(scope="module")
def handles():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hs = {k: F.ftgemm_create(v[0], 0) for k, v in KINDS.items()}
    yield hs
    for h in hs.values():
        F.ftgemm_destroy(h)


def _padded(X, ld, offset, nan):
    """X column-major with leading dimension ld, `offset` elements into a buffer whose padding is NaN."""
    import torch
    m, n = X.shape
    buf = np.full(offset + ld * n, nan, X.dtype)
    buf[offset:].reshape(n, ld)[:, :m] = X.T
    d = torch.from_numpy(buf.view(np.uint8)).cuda()
    return d, d.data_ptr() + X.itemsize * offset


def _run(h, kind, A, B, level, pad=(0, 0), offset=0):
    import torch
    nan = KINDS[kind][4]
    (m, k), n = A.shape, B.shape[1]
    dA, pA = _padded(A, m + pad[0], offset, nan)
    dB, pB = _padded(B, k + pad[1], offset, nan)
    dC = torch.zeros((n, m), device="cuda")
    rep = F.ReportBuffer(64)
    st = F.ftgemm_run(h, m, n, k, 1.0, pA, m + pad[0], pB, k + pad[1], 0.0, dC.data_ptr(), m, level, 0.0,
                      torch.cuda.current_stream().cuda_stream, rep)
    return st, dC.cpu().numpy().T, rep


def _operands(kind, m, n, k, seed):
    _, quantize, decode, dtype, _ = KINDS[kind]
    r = np.random.default_rng(seed)
    A, sa = quantize(r.standard_normal((m, k)).astype(np.float32))
    B, sb = quantize(r.standard_normal((k, n)).astype(np.float32))
    A, B = np.asarray(A).astype(dtype), np.asarray(B).astype(dtype)
    return A, B, np.asarray(decode(A), np.float64), np.asarray(decode(B), np.float64)


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("cfg", CONFIGS)
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 9), (6, 1, 33), (127, 130, 63), (129, 126, 64),
                                   (131, 257, 65), (254, 3, 191), (257, 255, 127), (256, 128, 256), (385, 130, 1)])
def test_edges(handles, kind, cfg, shape):
    m, n, k = shape
    A, B, a, b = _operands(kind, m, n, k, m * 7 + n * 3 + k)
    bound = _u(k) * (np.abs(a) @ np.abs(b)) + 2.0 ** -149
    F.ftgemm_set_config(handles[kind], cfg)
    try:
        for level in (0, 1, 2):
            for pad, offset in (((0, 0), 0), ((1, 3), 1), ((2, 5), 3)):
                st, C, rep = _run(handles[kind], kind, A, B, level, pad, offset)
                assert st == F.OK and rep.report.n_events == 0
                assert np.max(np.abs(C - a @ b) / bound) <= 1.0
    finally:
        F.ftgemm_set_config(handles[kind], None)


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("cfg", CONFIGS)
def test_faults_in_every_block(handles, kind, cfg):
    """One fault per 32 x 32 block of a full tile, each in a call of its own k-steps: located and corrected."""
    t = cfg[0]
    m = n = t
    k = 2 * 64 * cfg[3]
    A, B, a, b = _operands(kind, m, n, k, 11)
    h = handles[kind]
    import torch
    F.ftgemm_set_config(h, cfg)
    try:
        for q in range(t // 32):
            row, col = 32 * q + (7 * q) % 32, (32 * (q * 3 % (t // 32)) + (5 * q + 3) % 32)
            sites = np.zeros(1, F.FAULT_DTYPE)
            sites["kstep"], sites["row"], sites["col"], sites["kind"], sites["payload"] = q % 8, row, col, F.FAULT_ADD, 1e6
            F.ftgemm_set_injection(h, sites)
            st, C, rep = _run(h, kind, A, B, 2)
            log = F.ftgemm_get_injection_log(h)
            assert st == F.OK and rep.report.corrected == 1 and len(log) == 1
            res, cls, n_grey, bad = replay_against_gpu(np.asfortranarray(a), np.asfortranarray(b), cfg, rep, log)
            assert bad == 0 and event_keys(rep.events) == event_keys(res.events)
            bound = _u(k) * (np.abs(a) @ np.abs(b))
            bound[row, col] += _u(k) * (np.abs(a[row]) @ np.abs(b)).sum()
            assert np.max(np.abs(C - a @ b) / bound) <= 1.0
    finally:
        F.ftgemm_set_injection(h, None)
        F.ftgemm_set_config(h, None)
