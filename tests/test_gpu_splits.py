"""Products whose column ranges follow the time model, and FP64 launches over
several column groups, against a plain FP64 product."""
import numpy as np
import pytest

from gpu_util import announce, ciq_module, torch_cuda
from oracle import kernels as okern

pytestmark = pytest.mark.gpu


# one chunk, one range per chunk, many ranges; widths around the 64-column
# groups and the remainder that keeps a launch of its own
@pytest.mark.parametrize("n,s", [(1, 1), (64, 2), (65, 64), (700, 65), (1024, 1), (1025, 96), (1500, 97), (2000, 128),
                                 (900, 200)])
@pytest.mark.parametrize("form", ["kernel_mvm", "resident"])
def test_fp64_product_shapes(n, s, form):
    """FP64 entries (1.6e-16 relative, products of positive entries) and sums
    of n terms in any order: n 2^-52 of |K||V| bounds every element."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(3 * n + s)
    x, v = rng.random((n, 3)), rng.standard_normal((n, s))
    announce(f"fp64 product shapes {form} n={n} s={s}")
    prob = ciq.Problem(torch.from_numpy(x).cuda(), "rbf", [0.3], 1.1, 0.02)
    fn = ciq.ciq_kernel_mvm if form == "kernel_mvm" else ciq.ciq_kernel_mvm_resident
    y = fn(prob, torch.from_numpy(v).cuda()).cpu().numpy()
    K = okern.kernel_matrix("rbf", x, [0.3], 1.1, 0.02)
    bound = max(n, 64) * 2.0 ** -52 * (np.abs(K) @ np.abs(v))
    assert np.all(np.abs(y - K @ v) <= bound)


def test_noalloc_limit_is_the_documented_one():
    """The scratch bound counts the documented ranges, whatever ranges run: the
    largest accepted FP32 request runs, and one more column is refused."""
    torch = torch_cuda()
    ciq = ciq_module()
    import paper_2006_11267_amd._lib as L
    n = 40_000
    x = torch.rand(n, 3, device="cuda")
    prob = ciq.Problem(x, "rbf", [0.3], 1.0, 0.1)
    announce("noalloc limit")
    accepted = []
    for s in range(1, 220):   # one range of 209 columns fills the scratch
        v = torch.ones((n, s), device="cuda")
        y = torch.empty((n, s), device="cuda")
        try:
            ciq.ciq_kernel_mvm_noalloc(prob, v, y)
        except L.CIQError as e:
            assert e.status == L.CIQ_EINVAL
            break
        accepted.append(s)
        assert torch.equal(y, ciq.ciq_kernel_mvm(prob, v))
    assert accepted and accepted[-1] < 209
