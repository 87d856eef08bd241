"""The low-rank products (block partials, their sum, the application in ranges
of r) at the edges of their tiles, through the calls that are made of them."""
import numpy as np
import pytest

from gpu_util import announce, ciq_module, colwise_rel, torch_cuda
from oracle import ciq as oc
from oracle import posterior as opost

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("t,n_obs,s", [(65, 128, 1), (63, 255, 16), (64, 256, 17), (130, 287, 32), (97, 385, 33),
                                       (200, 520, 64), (129, 513, 65)])
def test_correction_in_ranges(t, n_obs, s):
    """Observation counts around one, two and four ranges of 32-row slabs,
    widths around the 16, 32 and 64 column tiles, candidates around 64 rows:
    FP64, fixed J, to 10x the oracle's own move when Sigma's entries move at
    the rounding scale of the two terms that it is the difference of."""
    torch = torch_cuda()
    ciq = ciq_module()
    d, J = 4, 4
    kind, ls, o2, jit, s2 = "matern52", [0.35], 1.0, 1e-2, 1e-2
    rng = np.random.default_rng(t + n_obs + s)
    xs, xo, b = rng.random((t, d)), rng.random((n_obs, d)), rng.standard_normal((t, s))
    S = opost.posterior_covariance(kind, xs, xo, ls, o2, jit, s2)
    Kss = opost.cross_kernel(kind, xs, xs, ls, o2)
    lam = np.linalg.eigvalsh(S)
    bounds = (lam[0], lam[-1])
    announce(f"low-rank ranges t={t} n_obs={n_obs} s={s}")
    prob = ciq.Problem(torch.from_numpy(xs).cuda(), kind, ls, o2, jit)
    out, info = ciq.ciq_posterior_mvm(prob, torch.from_numpy(xo).cuda(), s2, torch.from_numpy(b).cuda(), mode="sqrt",
                                      q=10, max_iter=J, tol=0.0, bounds=bounds)
    ref, _ = oc.ciq(lambda v: S @ v, b, bounds[0], bounds[1], 10, J, 0.0, "sqrt")
    assert info["iters"] == J
    mag = np.abs(Kss) + np.abs(Kss + jit * np.eye(t) - S)
    spread = 0.0
    for seed in range(2):
        E = np.random.default_rng(50 + seed).standard_normal(S.shape)
        Sp = S + 2.2e-16 * mag * (E + E.T) / np.sqrt(2.0)
        alt, _ = oc.ciq(lambda v: Sp @ v, b, bounds[0], bounds[1], 10, J, 0.0, "sqrt")
        spread = max(spread, colwise_rel(alt, ref).max())
    bar = max(10.0 * spread, 1e-11)
    gap = colwise_rel(out.cpu().numpy(), ref).max()
    print(f"gap {gap:.2e} bar {bar:.2e}", flush=True)
    assert gap < bar


@pytest.mark.parametrize("M,nb", [(16, 32), (17, 33), (33, 64), (65, 31), (129, 66)])
def test_rank_update_widths(M, nb):
    """The natural-gradient update's Theta is one application of rank nb and
    width M: widths in the narrow and wide tiles, even (16-byte rows) and odd
    ranks around a 32-row slab. 1e-12 of the largest entry (sums in another
    order of nb FP64 terms)."""
    torch = torch_cuda()
    ciq = ciq_module()
    rng = np.random.default_rng(M + nb)
    G = rng.standard_normal((M, M))
    Theta = -(G @ G.T / M + np.eye(M)) * 0.5
    theta = rng.standard_normal(M)
    a = rng.standard_normal((M, nb)) / np.sqrt(M)
    mean, cm, cv = rng.standard_normal(nb), rng.standard_normal(nb), -np.abs(rng.standard_normal(nb))
    from oracle import svgp as osv
    announce(f"low-rank update M={M} nb={nb}")
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).cuda()
    th, Th = dev(theta), dev(Theta)
    ciq.ciq_svgp_ngd_step(dev(a), dev(mean), dev(cm), dev(cv), th, Th, 37.0, 0.3)
    th_o, Th_o = osv.ngd_step(theta, Theta, a, mean, cm, cv, 37.0, 0.3)
    assert np.abs(Th.cpu().numpy() - Th_o).max() <= 1e-12 * np.abs(Th_o).max()
    assert np.abs(th.cpu().numpy() - th_o).max() <= 1e-12 * np.abs(th_o).max()
