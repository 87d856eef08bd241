"""The step after the product: one launch (small problems) or several, with
right-hand sides padded to a multiple of four columns, against the oracle."""
import numpy as np
import pytest

from gpu_util import announce, ciq_module, colwise_rel, torch_cuda
from oracle import ciq as ociq
from oracle import kernels as okern

pytestmark = pytest.mark.gpu


# around the one-launch step's limits (1024 rows; 8192 elements for one or two
# columns), its register rows (1, 2, 4, 8 a thread) and the padded widths
@pytest.mark.parametrize("n,s", [(2, 1), (255, 3), (513, 5), (1024, 6), (1025, 6), (1024, 64), (700, 66), (1600, 130),
                                 (1024, 2), (4096, 2), (4097, 2), (1025, 1), (8192, 1), (8193, 1)])
@pytest.mark.parametrize("basis", ["auto", "off"])
def test_step_small_j_parity(n, s, basis):
    """FP64, six iterations of a well-conditioned problem with given bounds:
    GPU and oracle agree to rounding (1e-11, the bar of the small-J parity
    tests); a zero column stays zero and does not disturb its neighbours."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(n * 131 + s)
    x, b = rng.random((n, 3)), rng.standard_normal((n, s))
    if s > 2:
        b[:, 1] = 0.0
    K = okern.kernel_matrix("matern52", x, [0.3], 1.0, 0.5)
    bounds = (0.5, 0.5 + 1.05 * n)
    J = min(6, n)
    announce(f"step parity n={n} s={s} basis={basis}")
    prob = ciq.Problem(torch.from_numpy(x).cuda(), "matern52", [0.3], 1.0, 0.5)
    out, info, _ = ciq.ciq_invsqrt_mvm(prob, torch.from_numpy(b).cuda(), q=9, max_iter=J, tol=0.0, bounds=bounds,
                                       krylov_basis=basis)
    live = [c for c in range(s) if np.any(b[:, c])]
    ref, oinfo = ociq.ciq(lambda v: K @ v, b[:, live], bounds[0], bounds[1], 9, J, 0.0, "invsqrt")
    got = out.cpu().numpy()
    assert info["iters"] == J and info["krylov_basis"] == (basis == "auto")
    assert colwise_rel(got[:, live], ref).max() < 1e-11
    if s > 2:
        assert np.all(got[:, 1] == 0.0)


@pytest.mark.parametrize("s", [1, 3, 5, 40])
def test_batched_step_widths(s):
    """Batched problems on both sides of the one-launch limit together (the
    largest decides) and alone, FP32: 1e-4 (the FP32 bar) against the dense
    root."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(s)
    for ns in ([1, 40, 333, 1024], [64, 900, 1500]):
        xs = [rng.random((n, 3)).astype(np.float32) for n in ns]
        bs = [rng.standard_normal((n, s)).astype(np.float32) for n in ns]
        announce(f"batched step widths s={s} ns={ns}")
        probs = [ciq.Problem(torch.from_numpy(x).cuda(), "rbf", [0.3], 1.0, 0.05) for x in xs]
        outs, infos = ciq.ciq_invsqrt_mvm_batched(probs, [torch.from_numpy(b).cuda() for b in bs], q=12, tol=1e-6)
        for x, b, o, i in zip(xs, bs, outs, infos):
            lam, U = np.linalg.eigh(okern.kernel_matrix("rbf", x.astype(np.float64), [0.3], 1.0, 0.05))
            ref = U @ ((U.T @ b.astype(np.float64)) / np.sqrt(lam)[:, None])
            assert i["converged"]
            assert colwise_rel(o.double().cpu().numpy(), ref).max() < 1e-4


# rows around the four a thread and the 16 a block, shifts around the 16 a
# launch, columns around the 64-column blocks and the padding
@pytest.mark.parametrize("n,s,q", [(1, 1, 3), (17, 2, 16), (63, 5, 17), (130, 65, 15), (1030, 3, 33)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_kept_solves_from_basis(n, s, q, prec):
    """Per-shift solves formed from the resident basis against dense shifted
    solves: FP64 run to 1e-12 relative residual (1e-9 of the solve: the
    residual over the smallest shifted eigenvalue, 0.5, times the 25-fold
    norm of this K), FP32 products 1e-4 (the FP32 bar). A zero column keeps
    zero solves."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(7 * n + s)
    dt = np.float64 if prec == "f64" else np.float32
    x, b = rng.random((n, 3)).astype(dt), rng.standard_normal((n, s)).astype(dt)
    if s > 2:
        b[:, 2] = 0.0
    K = okern.kernel_matrix("rbf", x.astype(np.float64), [0.2], 1.0, 0.5)
    announce(f"kept solves n={n} s={s} q={q} {prec}")
    prob = ciq.Problem(torch.from_numpy(x).cuda(), "rbf", [0.2], 1.0, 0.5)
    out, info, solves = ciq.ciq_invsqrt_mvm(prob, torch.from_numpy(b).cuda(), q=q, max_iter=500,
                                            tol=1e-12 if prec == "f64" else 1e-6, keep_solves=True)
    assert info["krylov_basis"] and info["converged"]
    live = [c for c in range(s) if np.any(b[:, c])]
    bar = 1e-9 if prec == "f64" else 1e-4
    acc = np.zeros((n, len(live)))
    for k in range(q):
        ref = np.linalg.solve(K + info["t"][k] * np.eye(n), b[:, live].astype(np.float64))
        got = solves[:, k, :].double().cpu().numpy()
        assert colwise_rel(got[:, live], ref).max() < bar
        if s > 2:
            assert np.all(got[:, 2] == 0.0)
        acc += info["w"][k] * ref
    assert colwise_rel(out.double().cpu().numpy()[:, live], acc).max() < bar
