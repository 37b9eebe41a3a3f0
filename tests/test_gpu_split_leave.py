"""GPU tests of what FP32 tiles on the three-way bf16 split do with operands
outside its range: which operands leave it (none for being small: the bits of a
product scaled by powers of two are those of the unscaled one), and what a
discarded pass leaves behind."""
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


def _ratio(C, A, B):
    """Largest element error in units of (k + 2) 2^-24 (|A||B|)_ij + k 2^-149 (one
    rounding per addition, also where the sums are denormal)."""
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    k = A.shape[1]
    return np.max(np.abs(C - A64 @ B64) / ((k + 2) * 2.0 ** -24 * (np.abs(A64) @ np.abs(B64)) + k * 2.0 ** -149))


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


@pytest.mark.parametrize("cfg", CONFIGS)
@pytest.mark.parametrize("value", [np.inf, np.nan, 3e30])
def test_events_of_a_discarded_pass(h, cfg, value):
    """A tolerance far below roundoff flags every check; the last k of one row
    takes its tiles off the split after two such checks.  Every check of a
    tile has one event, and its counts are those of the events."""
    m, n, k = 300, 270, 600
    A, B = _operands(m, n, k, 33)
    A[290, 597] = value
    st, C, rep, _ = _run(h, A, B, 2, tol=1e-6, cfg=cfg)
    keys = [(int(e["tile_m"]), int(e["tile_n"]), int(e["kstep"])) for e in rep.events]
    assert len(keys) == len(set(keys))
    tiles = ((m + cfg[0] - 1) // cfg[0]) * ((n + cfg[1] - 1) // cfg[1])
    assert rep.report.checks == 3 * tiles == len(keys)      # k-steps 7, 15 and 18 of 19
    kinds = [int(e["kind"]) for e in rep.events]
    assert rep.report.detected == len(kinds) - kinds.count(F.EV_NONFINITE)
    assert rep.report.uncorrectable == kinds.count(F.EV_UNCORRECTABLE)


@pytest.mark.parametrize("cfg", CONFIGS)
@pytest.mark.parametrize("level", [0, 1, 2])
@pytest.mark.parametrize("ea, eb", [(-103, 30), (-106, 30), (-109, 30), (-112, 30), (-118, 36), (-125, 30), (30, -112),
                                    (-20, -90), (36, -30), (-60, -40)])
def test_scaled_operands_keep_their_bits(h, cfg, level, ea, eb):
    """Full 24-bit mantissas times powers of two: no element leaves the split
    for being small, so the product's bits are the unscaled one's.  (The first
    32 k add exact zeros and give every line an ordinary norm.)"""
    m, n, k = 200, 140, 150
    r = np.random.default_rng(34)
    A = ((1 + r.random((m, k))) * r.choice([-1, 1], (m, k))).astype(np.float32)
    B = ((1 + r.random((k, n))) * r.choice([-1, 1], (k, n))).astype(np.float32)
    B[:16], A[:, 16:32] = 0.0, 0.0
    C = {}
    for sa, sb in ((0, 0), (ea, eb)):
        X, Y = A.copy(), B.copy()
        X[:, 32:] *= np.float32(2.0 ** sa)
        Y[32:] *= np.float32(2.0 ** sb)
        st, c, rep, _ = _run(h, X, Y, level, cfg=cfg)
        assert st == F.OK and rep.report.n_events == 0
        C[sa] = np.ldexp(c.astype(np.float64), -sa - sb)
    assert _ratio(C[0], A, B) <= 1.0
    assert np.array_equal(C[0], C[ea])


@pytest.mark.parametrize("cfg", CONFIGS)
@pytest.mark.parametrize("level", [0, 1, 2])
@pytest.mark.parametrize("scale", [2.0 ** -103, 2.0 ** -109, 2.0 ** -118, 2.0 ** -126, 2.0 ** -140])
def test_small_among_ordinary(h, cfg, level, scale):
    """Rows of ordinary norm whose products come from their small elements only, down to denormals."""
    m, n, k = 300, 140, 70
    A, B = _operands(m, n, k, 35)
    B[:35, :] = 0.0
    A[:, 35:] *= np.float32(scale)
    B[35:, :] *= np.float32(2.0 ** 30)
    st, C, rep, _ = _run(h, A, B, level, cfg=cfg)
    assert st == F.OK and rep.report.n_events == 0 and _ratio(C, A, B) <= 1.0


@pytest.mark.parametrize("cfg", CONFIGS)
@pytest.mark.parametrize("level", [0, 2])
@pytest.mark.parametrize("e", [-62, -66, -70])
def test_products_below_the_normal_range(h, cfg, level, e):
    A, B = _operands(256, 130, 64, 36)
    A, B = A * np.float32(2.0 ** e), B * np.float32(2.0 ** e)
    st, C, rep, _ = _run(h, A, B, level, cfg=cfg)
    assert st == F.OK and rep.report.n_events == 0 and _ratio(C, A, B) <= 1.0


@pytest.mark.parametrize("cfg", CONFIGS)
@pytest.mark.parametrize("k", [4, 16, 17, 18, 25, 31, 32, 33])
def test_short_positive_sums(h, cfg, k):
    """Sums of one sign over a few k, where the partial products round in one direction the most:
    the 2-norm error stays below that of a chain of K additions (an error of 2^-24 / sqrt(3) of each of the sums,
    which grow like i / K: sqrt(K / 9) 2^-24 in all) and a rounding of the result."""
    r = np.random.default_rng(k)
    A, B = r.random((256, k)).astype(np.float32), r.random((k, 256)).astype(np.float32)
    st, C, rep, _ = _run(h, A, B, 2, cfg=cfg)
    P = A.astype(np.float64) @ B.astype(np.float64)
    assert st == F.OK and np.linalg.norm(C - P) / np.linalg.norm(P) <= (np.sqrt(k / 9.0) + 1.0) * 2.0 ** -24


@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("tile", [256, 128])
def test_recomputed_tile_has_the_bits_of_a_clean_call(dtype, tile):
    import torch
    m, n, k = 300, 280, 512
    cfg = (tile, tile, 32 if dtype == "f32" else 64, 8 if dtype == "f32" else 4)
    g = torch.Generator(device="cuda").manual_seed(37)
    tt = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}[dtype]
    dA = torch.randn((k, m), generator=g, device="cuda").to(tt)
    dB = torch.randn((n, k), generator=g, device="cuda").to(tt)
    handle = F.ftgemm_create({"f32": F.F32, "bf16": F.BF16, "fp8": F.F8E4M3}[dtype], 0)
    out = []
    try:
        F.ftgemm_set_config(handle, cfg)
        for faulty in (False, True):
            dC = torch.zeros((n, m), device="cuda")
            sites = np.zeros(4, F.FAULT_DTYPE)      # two faults in one interval of the first and the last tile
            last_m, last_n = (m - 1) // tile, (n - 1) // tile
            sites["tile_m"], sites["tile_n"] = (0, 0, last_m, last_m), (0, 0, last_n, last_n)
            sites["kstep"], sites["row"], sites["col"] = (1, 2, 0, 1), (5, 20, 3, 7), (7, 17, 2, 9)
            sites["kind"], sites["payload"] = F.FAULT_ADD, 1e5
            F.ftgemm_set_injection(handle, sites if faulty else None)
            rep = F.ReportBuffer(64)
            st = F.ftgemm_run(handle, m, n, k, 1.0, dA.data_ptr(), m, dB.data_ptr(), k, 0.0, dC.data_ptr(), m,
                              F.FT_CORRECT | F.FT_RECOMPUTE, 0.0, torch.cuda.current_stream().cuda_stream, rep)
            assert st == F.OK and rep.report.recomputed == (2 if faulty else 0) and rep.report.recompute_failed == 0
            out.append(dC.cpu().numpy())
    finally:
        F.ftgemm_set_injection(handle, None)
        F.ftgemm_destroy(handle)
    assert np.array_equal(out[0], out[1])
