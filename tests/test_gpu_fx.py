"""FP32 products with entries evaluated in the product, more than 16 columns
(split entries on the BF16 matrix cores), through ciq_kernel_mvm and the solves
that evaluate entries."""
import numpy as np
import pytest

from gpu_util import announce, ciq_module, colwise_rel, torch_cuda
from oracle import ciq as oc
from oracle import kernels as okern

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,d,s,ls", [
    ("matern52", 1, 6, 17, [0.3]),                    # less than one tile
    ("rbf", 17, 2, 32, [0.4]),
    ("matern52", 63, 3, 33, [0.1, 0.4, 0.9]),
    ("rbf", 64, 4, 64, [0.3]),                        # one chunk, one sign
    ("matern52", 65, 5, 65, [0.5]),
    ("rbf", 127, 7, 48, [0.5] * 3 + [0.9] * 4),
    ("matern52", 129, 9, 127, [0.5]),
    ("rbf", 1000, 12, 128, [0.7]),
    ("matern52", 1029, 16, 129, [0.4] * 8 + [1.5] * 8),   # a last group of one column
    ("rbf", 2051, 6, 150, [0.02]),                    # next to the identity
    ("matern52", 4100, 6, 24, [0.3]),
])
def test_split_product(kind, n, d, s, ls):
    """Against float64 on the same points. An FP32 entry is off by the rounding
    of its squared distance (d + 2 roundings of 2^-24, halved by Matern's
    square root), times its exponent's slope t e^-t <= 1/e (RBF) or the like,
    and of the exponential (2 ulp); a sum of 64 columns rounds a few times:
    (d + 10) 2^-23 of |K| |v| bounds each element, and the dropped terms are far
    below. Rows of columns scaled by 1e-30 and 1e30 check the range."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(n + s)
    x = rng.random((n, d)).astype(np.float32)
    v = rng.standard_normal((n, s)).astype(np.float32)
    v[:, 0] *= np.float32(1e-30)
    v[:, 1] *= np.float32(1e30)
    announce(f"split on-the-fly product {kind} n={n} d={d} s={s}")
    prob = ciq.Problem(torch.from_numpy(x).cuda(), kind, ls, 1.3, 1e-2)
    y = ciq.ciq_kernel_mvm(prob, torch.from_numpy(v).cuda(), precision="f32").cpu().numpy().astype(np.float64)
    K = okern.kernel_matrix(kind, x.astype(np.float64), ls, 1.3, 1e-2)
    ref = K @ v.astype(np.float64)
    bound = (d + 10) * 2.0 ** -23 * (np.abs(K) @ np.abs(v.astype(np.float64)))
    worst = (np.abs(y - ref) / bound).max()
    print(f"worst element at {worst:.3f} of its bound", flush=True)
    assert worst < 1.0


def test_split_product_infinities_and_nan():
    """An infinite element reaches every row of its column with its sign, two of
    opposite sign and a NaN make the column NaN, the other columns stay as they
    were; elements that round up to infinity in 16 bits stay finite."""
    torch = torch_cuda()
    ciq = ciq_module()
    n, s = 200, 20
    rng = np.random.default_rng(0)
    x = torch.from_numpy(rng.random((n, 3)).astype(np.float32)).cuda()
    v = torch.from_numpy(rng.standard_normal((n, s)).astype(np.float32)).cuda()
    big = torch.finfo(torch.float32).max
    prob = ciq.Problem(x, "matern52", [2.0], 1.0, 1e-2)
    announce("split on-the-fly product: infinities")
    base = ciq.ciq_kernel_mvm(prob, v, precision="f32")
    w = v.clone()
    w[70, 0] = float("inf")
    w[3, 1] = float("-inf")
    w[5, 2], w[130, 2] = float("inf"), float("-inf")
    w[199, 3] = float("nan")
    w[:, 4] = 0.0
    w[64, 4] = big
    y = ciq.ciq_kernel_mvm(prob, w, precision="f32")
    assert bool((y[:, 0] == float("inf")).all()) and bool((y[:, 1] == float("-inf")).all())
    assert bool(torch.isnan(y[:, 2]).all()) and bool(torch.isnan(y[:, 3]).all())
    other = torch.arange(n, device=y.device) != 64        # row 64: (1 + noise) max overflows
    assert bool(torch.isfinite(y[other, 4]).all()) and float(y[other, 4].min()) > 0.0
    assert torch.equal(y[:, 5:], base[:, 5:])


@pytest.mark.parametrize("s,ldv", [(40, 41), (17, 64)])
def test_split_product_strided(s, ldv):
    """Columns of a wider row-major block, odd leading dimension: the contiguous
    copy's bits."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(s)
    x = torch.from_numpy(rng.random((777, 5)).astype(np.float32)).cuda()
    wide = torch.from_numpy(rng.standard_normal((777, ldv)).astype(np.float32)).cuda()
    prob = ciq.Problem(x, "rbf", [0.4], 1.0, 1e-2)
    announce(f"split on-the-fly product strided s={s} ld={ldv}")
    a = ciq.ciq_kernel_mvm(prob, wide[:, :s], precision="f32")
    b = ciq.ciq_kernel_mvm(prob, wide[:, :s].contiguous(), precision="f32")
    assert torch.equal(a, b)


@pytest.mark.parametrize("mode", ["sqrt", "invsqrt"])
def test_on_the_fly_solve(mode):
    """A converged root whose products evaluate entries (kernel_cache off) takes
    the split form at 48 columns; against the oracle to the tolerance of the
    other FP32 forms (1e-4 at this conditioning)."""
    torch = torch_cuda()
    ciq = ciq_module()
    n, s = 1500, 48
    rng = np.random.default_rng(4)
    x = rng.random((n, 4)).astype(np.float32)
    b = rng.standard_normal((n, s)).astype(np.float32)
    K = okern.kernel_matrix("matern52", x.astype(np.float64), [0.3], 1.0, 5e-2)
    lam = np.linalg.eigvalsh(K)
    announce(f"on-the-fly FP32 solve {mode}")
    prob = ciq.Problem(torch.from_numpy(x).cuda(), "matern52", [0.3], 1.0, 5e-2)
    fn = ciq.ciq_sqrt_mvm if mode == "sqrt" else ciq.ciq_invsqrt_mvm
    out, info, _ = fn(prob, torch.from_numpy(b).cuda(), q=12, max_iter=800, tol=5e-6, bounds=(lam[0], lam[-1]),
                      precision="f32", kernel_cache="off")
    assert info["converged"] and not info["kernel_cached"]
    ref, _ = oc.ciq(lambda u: K @ u, b.astype(np.float64), lam[0], lam[-1], 12, 2000, 1e-10, mode)
    err = colwise_rel(out.cpu().numpy().astype(np.float64), ref).max()
    print(f"{mode}: {err:.2e}, {info['iters']} iterations", flush=True)
    assert err < 1e-4
