"""The wide resident FP32 product (more than 32 columns, three-part FP16
splits) against a plain FP64 product of the same points."""
import numpy as np
import pytest

from gpu_util import announce, ciq_module, torch_cuda
from oracle import kernels as okern

pytestmark = pytest.mark.gpu


# rows around the 64-column chunks and the 128 / 256-row blocks, columns around
# the 16-column blocks, the three- and four-block groups and one to three groups
@pytest.mark.parametrize("n,s", [(1, 33), (63, 48), (129, 49), (257, 64), (640, 65), (1000, 97), (1281, 129),
                                 (2049, 160)])
@pytest.mark.parametrize("kind,scale", [("matern52", 1.0), ("rbf", 1e-18)])
def test_wide_fp32_product(n, s, kind, scale):
    """Entries are rounded once to FP32 (relative 2^-24 each, all positive) and
    the FP32 sums of 64 columns add a few 2^-24 of the column sums of |K||V|:
    4 x 2^-24 of |K||V| bounds every element. Right-hand sides far from 1 are
    scaled per column by a power of two, so the bound does not depend on them."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(n + s)
    x = rng.random((n, 5)).astype(np.float32)
    v = (rng.standard_normal((n, s)) * scale).astype(np.float32)
    v[:, 0] = 0.0
    announce(f"wide fp32 product n={n} s={s} {kind} scale={scale:g}")
    prob = ciq.Problem(torch.from_numpy(x).cuda(), kind, [0.4], 1.3, 0.05)
    y = ciq.ciq_kernel_mvm_resident(prob, torch.from_numpy(v).cuda()).double().cpu().numpy()
    K = okern.kernel_matrix(kind, x.astype(np.float64), [0.4], 1.3, 0.05)
    bound = 4.0 * 2.0 ** -24 * (np.abs(K) @ np.abs(v.astype(np.float64)))
    assert np.all(np.abs(y - K @ v.astype(np.float64)) <= bound + 1e-300)
    assert np.all(y[:, 0] == 0.0)


@pytest.mark.parametrize("s", [40, 130])
def test_wide_fp32_backward_sqrt(s):
    """The square root's backward starts from K G by the same product: dB for
    tol 1e-7 against the dense adjoint K^{1/2} G (2e-5: the FP32 entries'
    rounding times the conditioning of this problem, as for the forward)."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(s)
    n = 300
    x = rng.random((n, 3)).astype(np.float32)
    b = rng.standard_normal((n, s)).astype(np.float32)
    g = rng.standard_normal((n, s)).astype(np.float32)
    announce(f"wide fp32 backward sqrt s={s}")
    prob = ciq.Problem(torch.from_numpy(x).cuda(), "matern52", [0.4], 1.0, 0.1)
    out, info, solves = ciq.ciq_sqrt_mvm(prob, torch.from_numpy(b).cuda(), q=12, max_iter=600, tol=1e-7,
                                         keep_solves=True)
    dB, *_ = ciq.ciq_backward(prob, torch.from_numpy(g).cuda(), info["t"], info["w"], solves, mode="sqrt",
                              max_iter=600, tol=1e-7)
    lam, U = np.linalg.eigh(okern.kernel_matrix("matern52", x.astype(np.float64), [0.4], 1.0, 0.1))
    root = lambda m: U @ (np.sqrt(lam)[:, None] * (U.T @ m.astype(np.float64)))  # noqa: E731
    for got, ref in ((out, root(b)), (dB, root(g))):
        err = np.linalg.norm(got.double().cpu().numpy() - ref, axis=0) / np.linalg.norm(ref, axis=0)
        assert err.max() < 2e-5
