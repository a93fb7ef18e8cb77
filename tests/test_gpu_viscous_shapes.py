"""The viscous (BR1) kernels on meshes that leave their last workgroups short, with every order
and flux, walls and farfield: residual and stage update against the oracle."""
import functools
import math

import numpy as np
import pytest
import torch

from oracle.dg import DG
from synthetic import fields, kuhn_cube

pytestmark = pytest.mark.gpu

from gpu_common import assert_parity, make_mesh, solver  # noqa: E402

FAR = (1.0, 0.5 * math.sqrt(1.4), 0.0, 0.0, 1.0)
TOL = {"fp64": 1e-12, "fp32": 1e-5}
MU = 0.02


@functools.lru_cache(maxsize=4)
def reference(kind, p, flux):
    # 540 elements: 36 groups of 16, the last of the eight shares holds one; one tetrahedron: 4
    # groups, four empty shares
    mesh = make_mesh("single") if kind == "single" else kuhn_cube(
        (6, 5, 3), periodic=(False, False, True), jitter=0.2, bump_height=0.05, shuffle_seed=2209, vid_seed=2210)
    dg = DG(p, mesh.elem_vid, mesh.elem_xyz, mesh.bface_vid, mesh.bface_tag, farfield_prim=FAR, flux=flux, mu=MU)
    U, U0 = (torch.from_numpy(fields.random_coefficients(mesh.n_elem, dg.Np, seed=s, scale=0.01)).float().double()
             for s in (61, 62))
    return mesh, dg, U, U0, dg.residual(U)


def copies_of(mesh, n):
    n_vert = int(mesh.elem_vid.max()) + 1
    shift = np.arange(n)[:, None, None] * n_vert
    many = kuhn_cube(1, periodic=(False, False, True))
    many.elem_vid = (mesh.elem_vid[None] + shift).reshape(-1, 4)
    many.elem_xyz = np.tile(mesh.elem_xyz, (n, 1, 1))
    many.bface_vid = (mesh.bface_vid[None] + shift).reshape(-1, 3)
    many.bface_tag = np.tile(mesh.bface_tag, n)
    return many


# 253 disjoint copies: 8540 groups, 4 past a multiple of 8, more than 256 CUs hold wavefronts of the
# update kernel, which then takes a second group
@pytest.mark.parametrize("kind,copies", [("single", 1), ("ragged", 1), ("ragged", 253)])
@pytest.mark.parametrize("flux", ["rusanov", "roe"])
@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_residual_and_stage(p, prec, flux, kind, copies):
    mesh, dg, U, U0, R = reference(kind, p, flux)
    s = solver(p, prec, copies_of(mesh, copies), farfield=FAR, mu=MU)
    s.set_flux(flux)
    Ui, U0i = (s.set_state(X.repeat(copies, 1, 1).cuda()) for X in (U, U0))
    nan = lambda: torch.full_like(Ui, float("nan"))  # noqa: E731
    got_r = s.get_state(s.residual(Ui, nan())).view(copies, *U.shape).cpu()
    got_s = s.get_state(s.rk_stage(Ui, U0i, nan(), 0.75, 1.0)).view(copies, *U.shape).cpu()
    s.sync()
    for k in {0, copies // 2, copies - 1}:
        assert_parity(dg, got_r[k], R, TOL[prec], label=f"{kind} p={p} {prec} {flux} residual")
        # relative to the residual part of the stage; its fp32 output is rounded at U's size too
        l2, el = 0.25 * dg.l2_norm(R), (0.25 * R).abs().amax((0, 2))
        assert_parity(dg, got_s[k], 0.75 * U0 + 0.25 * (U + R), TOL[prec], l2_scale=l2, elem_scale=el,
                      label=f"{kind} p={p} {prec} {flux} stage")
    for got in (got_r, got_s):
        assert (got - got[:1]).abs().max() <= TOL[prec] * got.abs().max()
