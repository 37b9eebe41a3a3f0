"""GPU test of reports over more handles than the page of pinned counter words
holds: every handle's reports are its own, with and without pinned words, in any
order of creation and destruction, and from several threads."""
import threading

import numpy as np
import pytest

from paper_2305_01024_amd import ftgemm as F

pytestmark = pytest.mark.gpu


def test_reports_of_many_handles():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sizes = [64 * (1 + q % 5) for q in range(70)]      # 70 handles, 64 slots
    A = torch.randn(320 * 320, device="cuda")
    B = torch.randn(320 * 320, device="cuda")
    C = [torch.zeros(320 * 320, device="cuda") for _ in sizes]
    handles = [F.ftgemm_create(F.F32, 0) for _ in sizes]
    try:
        for h in handles:
            F.ftgemm_set_config(h, (64, 64, 32, 1000))

        def call(q):
            n = sizes[q]
            rep = F.ReportBuffer(16)
            st = F.ftgemm_run(handles[q], n, n, n, 1.0, A.data_ptr(), n, B.data_ptr(), n, 0.0, C[q].data_ptr(), n,
                              F.FT_CORRECT, 0.0, torch.cuda.current_stream().cuda_stream, rep)
            return st, rep.report.checks, rep.report.n_events

        def all_reports():
            for q in range(len(sizes)):
                assert call(q) == (F.OK, (sizes[q] // 64) ** 2, 0)      # one check per 64 x 64 tile

        all_reports()
        for q in range(0, 60, 3):       # slots given back and taken again
            F.ftgemm_destroy(handles[q])
            handles[q] = F.ftgemm_create(F.F32, 0)
            F.ftgemm_set_config(handles[q], (64, 64, 32, 1000))
        all_reports()

        wrong = []

        def worker(start):
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(20):
                    for q in range(start, len(sizes), 4):
                        if call(q) != (F.OK, (sizes[q] // 64) ** 2, 0):
                            wrong.append(q)

        threads = [threading.Thread(target=worker, args=(t,)) for t in range(4)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not wrong
    finally:
        for h in handles:
            F.ftgemm_destroy(h)
    h = F.ftgemm_create(F.F32, 0)       # the page was given back and is taken anew
    try:
        rep = F.ReportBuffer(4)
        F.ftgemm_run(h, 64, 64, 64, 1.0, A.data_ptr(), 64, B.data_ptr(), 64, 0.0, C[0].data_ptr(), 64, F.FT_CORRECT, 0.0,
                     torch.cuda.current_stream().cuda_stream, rep)
        assert rep.report.checks >= 1
    finally:
        F.ftgemm_destroy(h)
    assert np.isfinite(C[0][:64 * 64].cpu().numpy()).all()
