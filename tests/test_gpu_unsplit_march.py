"""Time marching and residual above every dispatch line of the stage kernel: eight disjoint copies of
a mesh (1,890 groups of 16 elements), each against the oracle on one."""
import functools
import math

import numpy as np
import pytest
import torch

from oracle.dg import DG
from synthetic import fields, kuhn_cube

pytestmark = pytest.mark.gpu

from gpu_common import assert_parity, solver  # noqa: E402

FAR = (1.0, 0.5 * math.sqrt(1.4), 0.0, 0.0, 1.0)
RESIDUAL_TOL = {"fp64": 1e-12, "fp32": 1e-5, "bf16": 5e-2, "fp16": 1e-2}
# increments are sums of residuals; FP32 rounds the state (2.6 against increments of 0.01) in six stages
STEP_TOL = {**RESIDUAL_TOL, "fp32": 1e-4}
COPIES, STEPS = 8, 2


@functools.lru_cache(maxsize=1)
def reference(p, flux):
    mesh = kuhn_cube((10, 9, 7), periodic=(False, False, True), jitter=0.2, bump_height=0.05, shuffle_seed=2209,
                     vid_seed=2210)
    dg = DG(p, mesh.elem_vid, mesh.elem_xyz, mesh.bface_vid, mesh.bface_tag, farfield_prim=FAR, flux=flux)
    U = torch.from_numpy(fields.random_coefficients(mesh.n_elem, dg.Np, seed=81, scale=0.01)).float().double()
    dt = 0.5 * dg.stable_dt(U)
    ref = U
    for _ in range(STEPS):
        ref = dg.rk3_step(ref, dt)
    return mesh, dg, U, dt, dg.residual(U), ref - U


# the reference's arguments vary slowest: one oracle run each
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16", "fp16"])
@pytest.mark.parametrize("flux", ["rusanov", "roe"])
@pytest.mark.parametrize("p", [1, 2, 3, 4])
def test_march_and_residual(p, flux, prec):
    mesh, dg, U, dt, R, inc = reference(p, flux)
    shift = np.arange(COPIES)[:, None, None] * (int(mesh.elem_vid.max()) + 1)
    many = kuhn_cube(1, periodic=(False, False, True))
    many.elem_vid = (mesh.elem_vid[None] + shift).reshape(-1, 4)
    many.elem_xyz = np.tile(mesh.elem_xyz, (COPIES, 1, 1))
    many.bface_vid = (mesh.bface_vid[None] + shift).reshape(-1, 3)
    many.bface_tag = np.tile(mesh.bface_tag, COPIES)
    s = solver(p, prec, many, farfield=FAR)
    s.set_flux(flux)
    assert s.n_elem_pad // 16 > 1536
    Ui = s.set_state(U.repeat(COPIES, 1, 1).cuda())
    got_r = s.get_state(s.residual(Ui, torch.full_like(Ui, float("nan")))).view(COPIES, *U.shape).cpu()
    # a work buffer of NaN bytes: a companion record or cell mean left unwritten would show
    work = s.new_work().fill_(255)
    s.rk_step(Ui, dt, STEPS, work)
    got = s.get_state(Ui).view(COPIES, *U.shape).cpu() - U
    s.sync()
    for k in (0, COPIES - 1):
        assert_parity(dg, got_r[k], R, RESIDUAL_TOL[prec], label=f"p={p} {prec} {flux} residual")
        assert_parity(dg, got[k], inc, STEP_TOL[prec], label=f"p={p} {prec} {flux} {STEPS} steps, increment")
    # the copies agree among themselves as far as two orders of summation do
    for x, tol in ((got_r, RESIDUAL_TOL), (got, STEP_TOL)):
        assert (x - x[:1]).abs().max() <= tol[prec] * x.abs().max()
