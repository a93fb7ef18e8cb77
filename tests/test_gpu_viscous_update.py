"""The viscous (BR1) path in FP32: what it holds in 64 bits."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from gpu_common import make_mesh, oracle, random_state, solver  # noqa: E402
from synthetic import fields, kuhn_cube  # noqa: E402


@pytest.mark.parametrize("p", [1, 2, 3, 4])
def test_fp32_update_takes_the_unrounded_residual(p):
    """The stage update is computed in fp64 from fp32 sums times an fp64 1/|K|; the residual is
    rounded to fp32 only where it is the output.  With U0 = -dt R, alpha = 1/2 and dt = 2^24 (both
    products exact) the stage gives (U + dt (R' - R)) / 2, where R' is the residual that the update
    took and |dt (R' - R)| is of the order of |R| unless R' is R, rounded.  The viscosity is
    negligible (1e-30), so that only the inviscid part counts."""
    mesh = make_mesh("ragged")
    dg = oracle(p, mesh)
    s = solver(p, "fp32", mesh, mu=1e-30)
    Ui = s.set_state(random_state(dg, seed=51).float().double().cuda())
    R = s.residual(Ui)
    dt = 2.0 ** 24
    out = s.get_state(s.rk_stage(Ui, -dt * R, s.new_state(), 0.5, dt))
    low = (2.0 * out - s.get_state(Ui)).abs()
    s.sync()
    R = s.get_state(R).abs()
    kept = (low[R > 0] > 0).double().mean().item()
    print(f"p={p}: {kept:.3f} of the entries carry bits below fp32")
    assert kept > 0.9
    # half an ulp of R, and the roundings of out (relative 2^-24 of at most |U| + |R|)
    assert (low <= R * (1 + 2.0 ** -20) + 2.0 ** -20).all()


def edges():
    """Two mesh widths h with h^2 exact in fp32, whose 1/|K| = 6 / h^3 fp32 rounds up and down by
    nearly half an ulp (relative 6e-8)."""
    m = np.float32(3.25) + np.arange(200000, dtype=np.float32) * np.float32(2.0 ** -22)
    m = m.astype(np.float64)
    iv = 6.0 / m ** 1.5
    d = iv.astype(np.float32).astype(np.float64) / iv - 1.0
    return np.sqrt(m[d.argmax()]), np.sqrt(m[d.argmin()]), d.max() - d.min()


@pytest.mark.parametrize("p", [1, 2, 3, 4])
def test_fp32_gradient_is_scaled_by_an_unrounded_volume(p):
    """Z = grad U is scaled by an fp64 1/|K| and rounded once.  A rounded 1/|K| scales all of Z, and
    with it the viscous residual, by the same wrong factor, which the projection of the FP32
    residual on the FP64 one shows: over thousands of entries their own roundings average out
    (about 1e-9), and so do the fp32 tables' when two mesh widths are compared."""
    c = []
    hi, lo, gap = edges()
    assert gap > 1.1e-7
    for h in (hi, lo):
        mesh = kuhn_cube(4, length=4.0 * h)
        U = torch.from_numpy(fields.random_coefficients(mesh.n_elem, oracle(p, mesh).Np, seed=52, scale=0.01))
        U = U.float().double().cuda()
        R = {}
        for prec in ("fp64", "fp32"):
            s = solver(p, prec, mesh, mu=1024.0, prandtl=0.875)  # kappa = 4096
            R[prec] = s.get_state(s.residual(s.set_state(U)))
            s.sync()
        c.append(((R["fp32"] * R["fp64"]).sum() / (R["fp64"] ** 2).sum()).item() - 1.0)
    print(f"p={p}: {c[0]:.2e} and {c[1]:.2e}")
    assert abs(c[0] - c[1]) < 2.0 ** -25
