"""One column of a sparse operator's solve (ciq_csr_mvm): the product that carries
the iteration's first inner product."""
import numpy as np
import pytest

from gpu_util import announce, ciq_module, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("n", [8192, 8193, 8255, 20033, 32768, 32769])
def test_csr_one_column_product_with_inner_product(n, graph):
    """Around the ends of the range in which one column's product carries the
    iteration's first inner product (and rows that do not fill its last block):
    a tridiagonal operator, converged, against its eigendecomposition (A = 2.5 I
    - shift - shift^T has sine eigenvectors), to 1e-8 at tol 1e-11 (16 nodes:
    1e-10 and better at this condition number of 9)."""
    torch = torch_cuda()
    ciq = ciq_module()
    from scipy.fft import dst, idst
    from scipy.sparse import diags
    A = diags([np.full(n - 1, -1.0), np.full(n, 2.5), np.full(n - 1, -1.0)], [-1, 0, 1], format="csr")
    lam = 2.5 - 2.0 * np.cos(np.pi * np.arange(1, n + 1) / (n + 1))
    b = np.random.default_rng(n).standard_normal((n, 1))
    announce(f"csr one column n={n} graph={graph}")
    csr = (torch.from_numpy(A.indptr.astype(np.int32)).cuda(), torch.from_numpy(A.indices.astype(np.int32)).cuda(),
           torch.from_numpy(A.data.astype(np.float64)).cuda())
    for mode, pw in (("invsqrt", -0.5), ("sqrt", 0.5)):
        out, info = ciq.ciq_csr_mvm(*csr, torch.from_numpy(b).cuda(), mode=mode, q=16, max_iter=500, tol=1e-11,
                                    bounds=(lam[0], lam[-1]), graph=graph)
        ref = idst(lam[:, None] ** pw * dst(b, type=1, axis=0), type=1, axis=0)
        err = np.linalg.norm(out.cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"n={n} {mode}: {err:.2e}, {info['iters']} iterations", flush=True)
        assert info["converged"] and err < 1e-8
