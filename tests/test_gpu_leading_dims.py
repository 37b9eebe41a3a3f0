"""GPU tests of leading dimensions just below and just past the 31-bit byte
offsets of the panel loads, for A and for B: the tile that cannot hold such an
offset leaves the operand to the general loads.  Operands are small integers,
so every sum is exact and the product has one value, whatever the order."""
import numpy as np
import pytest

from paper_2305_01024_amd import ftgemm as F

pytestmark = pytest.mark.gpu
# type: element bytes, k of a panel of the tile's loads, k-step of the interface
KINDS = {"f32": (4, 16, 32), "bf16": (2, 64, 64), "fp8": (1, 64, 64)}


@pytest.mark.parametrize("dtype", list(KINDS))
@pytest.mark.parametrize("operand", ["A", "B"])
@pytest.mark.parametrize("past", [False, True])
def test_leading_dimension_past_the_offsets(dtype, operand, past):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    es, panel, kstep = KINDS[dtype]
    tile = 128
    m, n, k = 140, (130 if operand == "A" else 5), (9 if operand == "A" else 100)
    limit = (1 << 31) // es // ((panel if operand == "A" else tile) + 1)
    ld = limit + (2 if past else -2)
    lda, ldb = (ld, k) if operand == "A" else (m, ld)
    tt = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}[dtype]
    g = torch.Generator(device="cuda").manual_seed(41)
    A = torch.randint(-3, 4, (k, m), generator=g, device="cuda").float().to(tt)      # column-major m x k
    B = torch.randint(-3, 4, (n, k), generator=g, device="cuda").float().to(tt)
    bits = {"f32": torch.int32, "bf16": torch.int16, "fp8": torch.int8}[dtype]
    bufA = torch.zeros((k - 1) * lda + m, device="cuda", dtype=bits)
    bufB = torch.zeros((n - 1) * ldb + k, device="cuda", dtype=bits)
    for c in range(k):
        bufA[c * lda:c * lda + m] = A[c].view(bits)
    for c in range(n):
        bufB[c * ldb:c * ldb + k] = B[c].view(bits)
    P = A.double().cpu().numpy().T @ B.double().cpu().numpy().T
    h = F.ftgemm_create({"f32": F.F32, "bf16": F.BF16, "fp8": F.F8E4M3}[dtype], 0)
    try:
        F.ftgemm_set_config(h, (tile, tile, kstep, 8))
        for level in (0, 2):
            C = torch.zeros((n, m), device="cuda")
            rep = F.ReportBuffer(64)
            st = F.ftgemm_run(h, m, n, k, 1.0, bufA.data_ptr(), lda, bufB.data_ptr(), ldb, 0.0, C.data_ptr(), m, level,
                              0.0, torch.cuda.current_stream().cuda_stream, rep)
            assert st == F.OK and rep.report.n_events == 0
            assert np.array_equal(C.cpu().numpy().T, P)
    finally:
        F.ftgemm_destroy(h)
