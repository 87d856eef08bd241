"""FP32 products of more than 32 columns against a resident matrix over the
range of FP32: very small columns, small entries and elements, infinities and
NaN."""
import numpy as np
import pytest

from gpu_util import announce, ciq_module, colwise_rel, torch_cuda
from oracle import kernels as okern

pytestmark = pytest.mark.gpu

TINY = 2.0 ** -119          # 1.5e-36: a normal FP32 number


def _case(torch, ciq, n, s, seed, kind="matern52", d=3, ls=0.4, noise=0.1, dense=True):
    rng = np.random.default_rng(seed)
    x = rng.random((n, d)).astype(np.float32)
    b = rng.standard_normal((n, s)).astype(np.float32)
    K = okern.kernel_matrix(kind, x.astype(np.float64), [ls], 1.0, noise) if dense else None
    return ciq.Problem(torch.from_numpy(x).cuda(), kind, [ls], 1.0, noise), b, K


@pytest.mark.parametrize("prec", ["f32", "f16x3"])
def test_tiny_column_product(prec):
    """A column scaled by 2^-119 is the unscaled column's product scaled: the
    operand's scale is a power of two per column (FP32 results of 2^-119 keep
    their 24 bits)."""
    torch = torch_cuda()
    ciq = ciq_module()
    prob, b, _ = _case(torch, ciq, 500, 40, 1)
    tiny = b.copy()
    tiny[:, 1] *= np.float32(TINY)
    b[:, 1] = tiny[:, 1] / TINY          # the same numbers: subnormal ones have lost bits
    announce(f"tiny column: resident product {prec}")
    y = ciq.ciq_kernel_mvm_resident(prob, torch.from_numpy(b).cuda(), precision=prec).cpu().numpy()
    yt = ciq.ciq_kernel_mvm_resident(prob, torch.from_numpy(tiny).cuda(), precision=prec).cpu().numpy()
    y[:, 1] *= np.float32(TINY)
    # elements below 2^-126 come out rounded to FP32's subnormal step
    assert np.all(np.abs(yt.astype(np.float64) - y) <= 2.0 ** -149)


@pytest.mark.parametrize("prec", ["f32", "f16x3"])
def test_tiny_column_roots(prec):
    """K^{1/2} B with a column of 2^-119 (its last product is with a vector that
    is not normalised), and the square root's backward (FP32; its first one is):
    against the dense FP64 result, 2e-5 per column in FP32 as in the other wide
    roots of this size, 1e-4 in split FP16."""
    torch = torch_cuda()
    ciq = ciq_module()
    prob, b, K = _case(torch, ciq, 300, 40, 2)
    b[:, 1] *= np.float32(TINY)
    lam, U = np.linalg.eigh(K)
    root = lambda m: U @ (np.sqrt(lam)[:, None] * (U.T @ m.astype(np.float64)))  # noqa: E731
    kw = dict(max_iter=600, tol=1e-7)
    announce(f"tiny column: square root and backward {prec}")
    bt = torch.from_numpy(b).cuda()
    out, info, _ = ciq.ciq_sqrt_mvm(prob, bt, q=12, precision=prec, kernel_cache="on", **kw)
    assert colwise_rel(out.cpu().numpy(), root(b)).max() < (2e-5 if prec == "f32" else 1e-4)
    if prec == "f32":
        _, info, solves = ciq.ciq_sqrt_mvm(prob, bt, q=12, keep_solves=True, **kw)
        dB, *_ = ciq.ciq_backward(prob, bt, info["t"], info["w"], solves, mode="sqrt", **kw)
        assert colwise_rel(dB.cpu().numpy(), root(b)).max() < 2e-5


@pytest.mark.parametrize("kind,ls", [("rbf", 0.1), ("matern52", 0.02)])
def test_small_entries(kind, ls):
    """Right-hand sides on four points only, short lengthscales: rows see them
    through entries down to FP32's smallest. Every entry is rounded once (2^-24),
    the operand to 2^-26, the dropped part products are 2^-25, four terms are cut
    off at 2^-23 at most and the result is rounded: 11 x 2^-24 of |K||V| bounds
    each element."""
    torch = torch_cuda()
    ciq = ciq_module()
    prob, v, K = _case(torch, ciq, 300, 40, 3, kind, d=5, ls=ls)
    v[4:] = 0.0
    announce(f"small entries {kind} ls={ls}")
    y = ciq.ciq_kernel_mvm_resident(prob, torch.from_numpy(v).cuda()).cpu().numpy().astype(np.float64)
    v = v.astype(np.float64)
    bound = 11 * 2.0 ** -24 * (np.abs(K) @ np.abs(v)) + 2.0 ** -148 * (1.0 + np.abs(v).sum(axis=0))
    worst = (np.abs(y - K @ v) / bound).max()
    print(f"worst element at {worst:.3f} of its bound", flush=True)
    assert worst < 1.0


def test_small_elements():
    """Next to the identity a row's result is its own element, however small
    beside the column's largest: elements from 1 to 2^-100, the bound as above
    (one term that counts)."""
    torch = torch_cuda()
    ciq = ciq_module()
    prob, v, K = _case(torch, ciq, 300, 40, 4, "rbf", d=5, ls=0.004)
    v = (np.sign(v) * 2.0 ** -np.minimum(np.arange(300) % 101, 100)[:, None] * (1.0 + np.abs(v) % 1.0)).astype(np.float32)
    announce("small elements")
    y = ciq.ciq_kernel_mvm_resident(prob, torch.from_numpy(v).cuda()).cpu().numpy().astype(np.float64)
    v = v.astype(np.float64)
    bound = 11 * 2.0 ** -24 * (np.abs(K) @ np.abs(v))
    assert (np.abs(y - K @ v) / bound).max() < 1.0


def test_sums_are_not_biased():
    """The matrix cores cut off downwards what an FP32 sum of eight products
    cannot hold, always with the same sign; signs that alternate from chunk to
    chunk cancel that. All positive sums: entries and results are rounded to
    nearest, 2^-25 each that averages out over 4,096 rows, so a mean signed
    relative error of 2^-26 would be the sums'."""
    torch = torch_cuda()
    ciq = ciq_module()
    prob, v, K = _case(torch, ciq, 4096, 40, 8, "matern52", d=6, ls=0.3, noise=1e-2)
    v = np.abs(v)
    announce("bias of the sums")
    y = ciq.ciq_kernel_mvm_resident(prob, torch.from_numpy(v).cuda()).cpu().numpy().astype(np.float64)
    ref = K @ v.astype(np.float64)
    bias = ((y - ref) / ref).mean() * 2.0 ** 26
    print(f"mean signed relative error {bias:.3f} x 2^-26", flush=True)
    assert abs(bias) < 1.0


def test_infinities_and_nan():
    """An infinite element reaches every row of its column with its sign, two of
    opposite sign and a NaN make the column NaN, a column with one element at
    FP32's end stays finite elsewhere, the other columns stay as they were."""
    torch = torch_cuda()
    ciq = ciq_module()
    n = 200
    prob, v, _ = _case(torch, ciq, n, 40, 5, ls=2.0)
    v = torch.from_numpy(v).cuda()
    announce("wide resident product: infinities")
    base = ciq.ciq_kernel_mvm_resident(prob, v)
    w = v.clone()
    w[70, 0] = float("inf")
    w[3, 1] = float("-inf")
    w[5, 2], w[130, 2] = float("inf"), float("-inf")
    w[199, 3] = float("nan")
    w[:, 4] = 0.0
    w[64, 4] = torch.finfo(torch.float32).max
    y = ciq.ciq_kernel_mvm_resident(prob, w)
    assert bool((y[:, 0] == float("inf")).all()) and bool((y[:, 1] == float("-inf")).all())
    assert bool(torch.isnan(y[:, 2]).all()) and bool(torch.isnan(y[:, 3]).all())
    other = torch.arange(n, device=y.device) != 64        # row 64: (1 + noise) max overflows
    assert bool(torch.isfinite(y[other, 4]).all()) and float(y[other, 4].min()) > 0.0
    assert torch.equal(y[:, 5:], base[:, 5:])


@pytest.mark.parametrize("mode", ["sqrt", "invsqrt"])
@pytest.mark.parametrize("basis", ["auto", "off"])
def test_wide_solve_basis_and_graph(mode, basis):
    """Wide resident solves with and without the Krylov basis (the operand is
    written by the update kernel of either) against the dense root, 1e-4 as for
    the other FP32 solves of this conditioning; graph replays (host polls between
    them) give the eager loop's bits."""
    torch = torch_cuda()
    ciq = ciq_module()
    prob, b, K = _case(torch, ciq, 1501, 41, 6, d=4, ls=0.3)
    lam, U = np.linalg.eigh(K)
    p = 0.5 if mode == "sqrt" else -0.5
    ref = U @ ((lam ** p)[:, None] * (U.T @ b.astype(np.float64)))
    fn = ciq.ciq_sqrt_mvm if mode == "sqrt" else ciq.ciq_invsqrt_mvm
    kw = dict(q=12, max_iter=800, tol=5e-6, bounds=(lam[0], lam[-1]), kernel_cache="on", krylov_basis=basis)
    announce(f"wide solve {mode} basis={basis}")
    bt = torch.from_numpy(b).cuda()
    out, info, _ = fn(prob, bt, **kw)
    assert info["converged"] and info["kernel_cached"] and info["krylov_basis"] == (basis == "auto")
    err = colwise_rel(out.cpu().numpy(), ref).max()
    print(f"{mode} basis={basis}: {err:.2e}, {info['iters']} iterations", flush=True)
    assert err < 1e-4
    for _ in range(2):
        g, ginfo, _ = fn(prob, bt, graph=True, **kw)
        assert ginfo["iters"] == info["iters"] and torch.equal(g, out)


def _fp64_inverse_root(torch, ciq, prob, b):
    """The same quadrature (its bounds returned) with FP64 products, converged."""
    p64 = ciq.Problem(prob.x.double(), prob.kernel, prob.lengthscale, prob.outputscale, prob.noise)
    ref, info, _ = ciq.ciq_invsqrt_mvm(p64, b.double(), q=15, max_iter=12000, tol=1e-10)
    assert info["converged"]
    return ref.cpu().numpy(), (info["lambda_min"], info["lambda_max"])


@pytest.mark.parametrize("cache", ["on", "off"])
@pytest.mark.parametrize("kind,n,d,ls,noise", [
    ("rbf", 4000, 3, 0.2, 1e-3),             # kappa 3e5
    ("rbf", 4000, 3, 0.2, 1e-2),
    ("matern52", 33000, 6, 0.3, 1e-2),       # 1.6e5
    ("matern52", 32700, 6, 0.3, 1e-1),
])
def test_wide_inverse_root_noise(kind, n, d, ls, noise, cache):
    """K^{-1/2} B of 40 columns: FP32 rounding of the products reaches the root
    multiplied by about kappa / sqrt(N). A resident product is off by at most 1.2
    x 2^-24 of its norm, one that evaluates FP32 entries by 2.5 x 2^-24 (their
    own rounding), at any conditioning and size; the solver's tolerance adds 1e-6."""
    torch = torch_cuda()
    ciq = ciq_module()
    prob, b, _ = _case(torch, ciq, n, 40, 9, kind, d=d, ls=ls, noise=noise, dense=False)
    bt = torch.from_numpy(b).cuda()
    announce(f"wide inverse root {kind} n={n} noise={noise} cache={cache}")
    ref, bounds = _fp64_inverse_root(torch, ciq, prob, bt)
    out, info, _ = ciq.ciq_invsqrt_mvm(prob, bt, q=15, max_iter=12000, tol=2e-7, bounds=bounds, kernel_cache=cache)
    err = colwise_rel(out.cpu().numpy(), ref).mean()
    unit = 2.0 ** -24 * bounds[1] / bounds[0] / np.sqrt(n)
    print(f"{kind} n={n} kappa={bounds[1] / bounds[0]:.2g} cache={cache}: {err:.2e} = {err / unit:.2f} units",
          flush=True)
    assert err < (1.2 if cache == "on" else 2.5) * unit + 1e-6


@pytest.mark.parametrize("kind,d,ls", [("rbf", 4, 0.35), ("matern52", 6, 0.3)])
def test_wide_sqrt_scalar_gradients(kind, d, ls):
    """Gradients of <G, K^{1/2} B> for the hyperparameters, whose sums cancel:
    against the same with FP64 products on the same quadrature, over six seeds, in
    units of the values' own size. The products' noise (2^-24) reaches the solves
    multiplied by kappa / sqrt(N) = 30; gradients for the lengthscale and the
    outputscale average it over N S terms, the noise's (a trace) is the smallest
    difference: 1e-5 of the first two, 1e-4 of the last."""
    torch = torch_cuda()
    ciq = ciq_module()
    n, s = 1000, 64
    errs, vals = [], []
    for seed in range(6):
        prob, b, _ = _case(torch, ciq, n, s, 100 + seed, kind, d=d, ls=ls, noise=5e-2, dense=False)
        bt = torch.from_numpy(b).cuda()
        g = torch.from_numpy(np.random.default_rng(seed).standard_normal((n, s)).astype(np.float32)).cuda()
        p64 = ciq.Problem(prob.x.double(), kind, [ls], 1.0, 5e-2)
        announce(f"scalar gradients {kind} seed={seed}")
        kw = dict(max_iter=2000)
        _, info, sol = ciq.ciq_sqrt_mvm(p64, bt.double(), q=15, tol=1e-11, keep_solves=True, **kw)
        ref = ciq.ciq_backward(p64, g.double(), info["t"], info["w"], sol, mode="sqrt", tol=1e-11, **kw)
        _, i32, sol = ciq.ciq_sqrt_mvm(prob, bt, q=15, tol=1e-7, keep_solves=True,
                                       bounds=(info["lambda_min"], info["lambda_max"]), **kw)
        got = ciq.ciq_backward(prob, g, i32["t"], i32["w"], sol, mode="sqrt", tol=1e-7, **kw)
        vals.append([float(np.ravel(ref[k])[0]) for k in (1, 2, 3)])
        errs.append([float(np.ravel(got[k])[0]) - vals[-1][k - 1] for k in (1, 2, 3)])
        assert colwise_rel(got[0].cpu().numpy(), ref[0].cpu().numpy()).max() < 1e-5
    rms = lambda a: np.sqrt((np.array(a) ** 2).mean(axis=0))  # noqa: E731
    rel = rms(errs) / rms(vals)
    print(f"{kind}: lengthscale {rel[0]:.1e}, outputscale {rel[1]:.1e}, noise {rel[2]:.1e}", flush=True)
    assert rel[0] < 1e-5 and rel[1] < 1e-5 and rel[2] < 1e-4
