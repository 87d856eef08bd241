"""Calls that fit in the device's memory by a little."""
import pytest

from gpu_util import announce, ciq_module, torch_cuda

pytestmark = pytest.mark.gpu


def test_three_columns_that_just_fit():
    """Three columns run as four where there is room. The direction recurrence
    holds 34 vectors (2 Lanczos, a product, 2 x 15 directions, the solution): 13.7
    GB for 2^24 rows of three columns, 18.3 GB for four. With 16 GiB left the call
    must run, as three; A is diagonal, so the result is known."""
    torch = torch_cuda()
    ciq = ciq_module()
    n, s = 1 << 24, 3
    announce("three columns that just fit")
    g = torch.Generator(device="cuda").manual_seed(1)
    diag = 1.0 + torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    b = torch.randn(n, s, generator=g, device="cuda", dtype=torch.float64)
    ptr = torch.arange(n + 1, device="cuda", dtype=torch.int32)
    col = torch.arange(n, device="cuda", dtype=torch.int32)
    out = torch.empty(n, s, device="cuda", dtype=torch.float64)
    del out                                              # (torch keeps it for the call)
    ciq.ciq_release_workspace()
    free, _ = torch.cuda.mem_get_info()
    fill = torch.empty(free - (16 << 30), dtype=torch.uint8, device="cuda")
    try:
        got, info = ciq.ciq_csr_mvm(ptr, col, diag, b, q=15, max_iter=100, tol=1e-9, bounds=(1.0, 2.0))
    finally:
        del fill
        torch.cuda.empty_cache()
        ciq.ciq_release_workspace()
    assert info["converged"] and not info["krylov_basis"]
    assert float((got - b / diag.sqrt()[:, None]).norm() / b.norm()) < 1e-7
