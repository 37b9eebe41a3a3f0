"""GPU tests of the FP32-output epilogue: tiles of whole and of ragged columns,
ragged rows, a C whose padding must stay, offsets of C, and a leading dimension
past the 32-bit offsets of the whole-column path.

Operands, alpha, beta and C are small integers, so every product and sum is
exact in FP32 whatever its order, and C must equal the integers."""
import numpy as np
import pytest

from paper_2305_01024_amd import ftgemm as F

pytestmark = pytest.mark.gpu
# e4m3 encodings of -2 .. 2
E4M3 = np.array([0xc0, 0xb8, 0x00, 0x38, 0x40], np.uint8)
KINDS = {"f32": F.F32, "bf16": F.BF16, "fp8": F.F8E4M3}
LARGE = {"f32": (256, 256, 32, 8), "bf16": (256, 256, 64, 4), "fp8": (256, 256, 64, 4)}
SHAPES = [(129, 256, 65), (256, 128, 33), (100, 64, 40), (257, 257, 64), (7, 512, 9), (300, 255, 130)]


def _operand(r, kind, m, n):
    import torch
    v = r.integers(-2, 3, (n, m))
    if kind == "fp8":
        return v.T, torch.from_numpy(E4M3[v + 2]).cuda()
    return v.T, torch.from_numpy(v.astype(np.float32)).cuda().to(torch.float32 if kind == "f32" else torch.bfloat16)


def _check(kind, m, n, k, ldc, offset, beta, level, cfg=None):
    import torch
    r = np.random.default_rng(m + 3 * n + 7 * k)
    A, dA = _operand(r, kind, m, k)
    B, dB = _operand(r, kind, k, n)
    flat = torch.empty(offset + ldc * n, device="cuda")
    C = flat[offset:].view(n, ldc)
    C[:, :m + 4] = 5.0 if beta else float("nan")
    C[:, m:m + 4] = float("nan")
    h = F.ftgemm_create(KINDS[kind], 0)
    try:
        F.ftgemm_set_config(h, cfg)
        st = F.ftgemm_run(h, m, n, k, 3.0, dA.data_ptr(), m, dB.data_ptr(), k, beta, C.data_ptr(), ldc, level, 0.0,
                          torch.cuda.current_stream().cuda_stream, F.ReportBuffer(16))
    finally:
        F.ftgemm_destroy(h)
    assert st == F.OK
    got = C[:, :m + 4].cpu().numpy()
    assert np.isnan(got[:, m:min(m + 4, ldc)]).all()
    assert np.array_equal(got[:, :m].T, 3.0 * (A @ B) + (5.0 * beta if beta else 0.0))


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("shape", SHAPES)
def test_exact(kind, shape):
    m, n, k = shape
    for beta in (0.0, -2.0):
        for level in (0, 2):
            for ldc, offset in ((m + 4, 0), (m + 5, 1)):
                for cfg in (None, LARGE[kind]):
                    _check(kind, m, n, k, ldc, offset, beta, level, cfg)


def test_leading_dimension_past_the_offsets():
    # (128 + 1) ldc 4 > 2^31: a 2.2 GB C of which 200 rows are written
    _check("f32", 200, 128, 40, 4200000, 0, -2.0, 2)
