"""FP32 products with entries evaluated in the product, more than 16 columns,
at the lower end of FP32's range."""
import numpy as np
import pytest

from gpu_util import announce, ciq_module, torch_cuda
from oracle import kernels as okern

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [20, 70])
def test_tiny_columns(s):
    """A column scaled by 2^-119 gives the unscaled column's result scaled, also
    where one of its elements is large; FP32's subnormal step apart."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(s)
    n = 500
    prob = ciq.Problem(torch.from_numpy(rng.random((n, 3)).astype(np.float32)).cuda(), "rbf", [0.4], 1.0, 0.1)
    b = rng.standard_normal((n, s)).astype(np.float32)
    tiny = b.copy()
    tiny[:, 1] *= np.float32(2.0 ** -119)
    tiny[:, 2] *= np.float32(2.0 ** -119)
    b[:, 1] = tiny[:, 1] / 2.0 ** -119     # the same numbers: subnormal ones have lost bits
    tiny[100, 2] = 0.0
    announce(f"tiny columns on the fly s={s}")
    y, yt = (ciq.ciq_kernel_mvm(prob, torch.from_numpy(v).cuda(), precision="f32").cpu().numpy().astype(np.float64)
             for v in (b, tiny))
    assert np.all(np.abs(yt[:, 1] - y[:, 1] * 2.0 ** -119) <= 2.0 ** -149)
    assert np.array_equal(yt[:, 0], y[:, 0]) and np.array_equal(yt[:, 3:], y[:, 3:])
    tiny[100, 2] = 1.0          # adds its own column of K to the one that is there
    y2 = ciq.ciq_kernel_mvm(prob, torch.from_numpy(tiny).cuda(), precision="f32").cpu().numpy().astype(np.float64)
    e = np.zeros((n, s), dtype=np.float32)
    e[100] = 1.0
    ye = ciq.ciq_kernel_mvm(prob, torch.from_numpy(e).cuda(), precision="f32").cpu().numpy().astype(np.float64)
    assert np.array_equal(y2[:, 2], ye[:, 2])


@pytest.mark.parametrize("kind,ls", [("rbf", 0.07), ("matern52", 0.02)])
def test_small_entries(kind, ls):
    """One right-hand side element, so that row i's result is its entry, as far
    as its exponential e^-x is a normal FP32 number. An FP32 entry is off by x
    times the relative error of its exponent ((d + 6) 2^-24: d + 3 for the squared
    distance, one each for the constant, the product and the square root) and by
    the exponential, the polynomial and the split products (8 x 2^-24)."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(7)
    n, d, s = 400, 3, 20
    x = rng.random((n, d)).astype(np.float32)
    v = np.zeros((n, s), dtype=np.float32)
    v[np.arange(s) * 19, np.arange(s)] = 1.0
    announce(f"small entries on the fly {kind}")
    prob = ciq.Problem(torch.from_numpy(x).cuda(), kind, [ls], 1.0, 0.1)
    y = ciq.ciq_kernel_mvm(prob, torch.from_numpy(v).cuda(), precision="f32").cpu().numpy().astype(np.float64)
    ref = okern.kernel_matrix(kind, x.astype(np.float64), [ls], 1.0, 0.1) @ v.astype(np.float64)
    r2 = okern.scaled_sqdist(x.astype(np.float64), x[np.arange(s) * 19].astype(np.float64), [ls] * d)
    expo = 0.5 * r2 if kind == "rbf" else np.sqrt(5.0 * r2)
    some = expo <= 125 * np.log(2.0)                     # the exponential is a normal FP32 number
    assert (expo[some] > 100 * np.log(2.0)).sum() > 50   # the range that is looked at
    rel = np.abs(y[some] - ref[some]) / ref[some]
    worst = (rel / ((expo[some] * (d + 6) + 8) * 2.0 ** -24)).max()
    print(f"worst element at {worst:.3f} of its bound", flush=True)
    assert worst < 1.0


def test_wide_range_of_elements():
    """Next to the identity a row's result is its own element: elements from 2^-120
    to 2^120 in one column, large ones (which take a pass of their own) and small
    ones in the same 64-row chunk. Entry and noise are exact there; the result is
    rounded once (2^-24) and float64 sums add nothing."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(11)
    n, s = 300, 40
    x = rng.random((n, 5)).astype(np.float32)
    v = (2.0 ** ((np.arange(n) * 37) % 241 - 120)[:, None] * rng.uniform(1, 2, (n, s))).astype(np.float32)
    v[:, 1] = np.abs(v[:, 1]) % 1.0                     # no large ones in this column
    announce("wide range of elements on the fly")
    prob = ciq.Problem(torch.from_numpy(x).cuda(), "rbf", [0.001], 1.0, 0.0)
    y = ciq.ciq_kernel_mvm(prob, torch.from_numpy(v).cuda(), precision="f32").cpu().numpy()
    ref = okern.kernel_matrix("rbf", x.astype(np.float64), [0.001], 1.0, 0.0)
    assert np.array_equal(ref, np.eye(n))
    assert np.array_equal(y, v)
