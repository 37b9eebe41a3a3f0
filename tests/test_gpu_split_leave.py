"""GPU tests of what FP32 tiles on the three-way bf16 split do with operands
outside its range: what a discarded pass leaves behind."""
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
    F.ftgemm_set_injection(handle, None)
    F.ftgemm_destroy(handle)


def _dev(X):
    import torch
    return torch.from_numpy(np.ascontiguousarray(X.T)).cuda()


def _run(h, A, B, level, tol=0.0, cfg=None, sites=None):
    import torch
    m, k = A.shape
    n = B.shape[1]
    dA, dB = _dev(A), _dev(B)
    dC = torch.zeros((n, m), device="cuda")
    rep = F.ReportBuffer(4096)
    F.ftgemm_set_config(h, cfg)
    F.ftgemm_set_injection(h, sites)
    try:
        st = F.ftgemm_run(h, m, n, k, 1.0, dA.data_ptr(), m, dB.data_ptr(), k, 0.0, dC.data_ptr(), m, level, tol,
                          torch.cuda.current_stream().cuda_stream, rep)
        log = F.ftgemm_get_injection_log(h) if sites is not None else None
    finally:
        F.ftgemm_set_injection(h, None)
        F.ftgemm_set_config(h, None)
    return st, dC.cpu().numpy().T.copy(), rep, log


def _operands(m, n, k, seed):
    r = np.random.default_rng(seed)
    return r.standard_normal((m, k)).astype(np.float32), r.standard_normal((k, n)).astype(np.float32)


def _faults(cfg, last):
    sites = np.zeros(2, F.FAULT_DTYPE)
    sites["tile_m"] = sites["tile_n"] = (0, last)
    sites["kstep"], sites["row"], sites["col"] = (1, 9), (17, 30), (40, 20)
    sites["kind"] = F.FAULT_ADD
    return sites


@pytest.mark.parametrize("cfg", CONFIGS)
@pytest.mark.parametrize("level", [0, 1, 2])
@pytest.mark.parametrize("size", [2.0 ** 40, 4e17, 1e18, 2.0 ** 62])
def test_faults_among_large_operands(h, cfg, level, size):
    """Elements of any size whose rows' squares pass the split's limit (and from
    1e18 on FP32's range): each fault is applied, and logged, once."""
    m = n = 300
    k = 512
    A, B = _operands(m, n, k, 31)
    A *= np.float32(size)
    last = (m - 1) // cfg[0]
    sites = _faults(cfg, last)
    sites["payload"] = np.float32(1e6) * np.float32(size)
    st, C, rep, log = _run(h, A, B, level, cfg=cfg, sites=sites)
    assert len(log) == 2
    assert sorted(map(int, log["tile_m"])) == [0, last]
    if level:
        assert all(int(x) >= 0 for x in log["check_step"])
    with np.errstate(over="ignore"):
        finite = np.isfinite(np.sum(A.astype(np.float32) ** 2, axis=1, dtype=np.float32)).all()
    if finite and level == 2:
        assert st == F.OK and rep.report.corrected == 2 and rep.report.n_events == 2
    elif finite and level == 1:
        assert rep.report.detected == 2 and rep.report.n_events == 2


@pytest.mark.parametrize("size", [4e17, 1e18])
def test_faults_among_large_operands_of_a_batch(h, size):
    import torch
    m, n, k = 200, 150, 512
    A, B = _operands(m, n, k, 32)
    A *= np.float32(size)
    dA, dB = _dev(A), _dev(B)
    dC = torch.zeros((n, m), device="cuda")
    probs = F.make_problems(1)
    probs[0] = (F.F32, 0, m, n, k, m, k, m, 1.0, 0.0, 1.0, 1.0, dA.data_ptr(), dB.data_ptr(), dC.data_ptr())
    sites = np.zeros(1, F.FAULT_DTYPE)
    sites["kstep"], sites["row"], sites["col"], sites["kind"], sites["payload"] = 1, 3, 5, F.FAULT_ADD, 1e6 * size
    rep = F.ReportBuffer(64)
    F.ftgemm_set_injection(h, sites)
    try:
        F.ftgemm_batched(h, probs, F.FT_CORRECT, 0.0, torch.cuda.current_stream().cuda_stream, rep)
        log = F.ftgemm_get_injection_log(h)
    finally:
        F.ftgemm_set_injection(h, None)
    assert len(log) == 1 and int(log["check_step"][0]) >= 0
