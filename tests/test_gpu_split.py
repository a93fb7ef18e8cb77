"""Both forms of the kernels that split a 16-element group over a workgroup on small meshes: a
ragged mesh below every dispatch line and one above (with walls, farfield and both fluxes),
against the oracle on sampled elements."""
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
TOL = {"fp64": 1e-12, "fp32": 1e-5, "bf16": 5e-2, "fp16": 1e-2}
SIZES = {"below": (10, 9, 7), "above": (17, 16, 17)}  # 237 and 1734 groups of 16 elements


@functools.lru_cache(maxsize=2)
def walls(size, p, flux):
    mesh = kuhn_cube(SIZES[size], periodic=(False, False, True), jitter=0.2, bump_height=0.05, shuffle_seed=2209,
                     vid_seed=2210)
    dg = DG(p, mesh.elem_vid, mesh.elem_xyz, mesh.bface_vid, mesh.bface_tag, farfield_prim=FAR, flux=flux)
    U, U0 = (torch.from_numpy(fields.random_coefficients(mesh.n_elem, dg.Np, seed=s, scale=0.01)) for s in (41, 42))
    # sampled elements, the mesh's last group (in the caller's order: any) among them
    sample = torch.from_numpy(np.sort(np.random.default_rng(5).choice(mesh.n_elem, 256, replace=False)))
    return mesh, dg, U, U0, sample, dg.residual(U, sample)


@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("size", ["below", "above"])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16", "fp16"])
def test_stage_both_sides_of_the_line(p, size, prec):
    """One stage with U0 (alpha = 3/4, dt = 1); the error is relative to its residual part."""
    mesh, dg, U, U0, sample, R = walls(size, p, "roe" if p % 2 else "rusanov")
    s = solver(p, prec, mesh, farfield=FAR)
    s.set_flux(dg.flux)
    out = s.get_state(s.rk_stage(s.set_state(U.cuda()), s.set_state(U0.cuda()), s.new_state(), 0.75, 1.0)).cpu()
    s.sync()
    if prec == "fp32":  # the stage inputs are stored in fp32
        U, U0 = U.float().double(), U0.float().double()
    ref = 0.75 * U0[sample] + 0.25 * (U[sample] + R)
    vol = dg.volume[sample]
    l2 = torch.sqrt((vol[:, None, None] * (0.25 * R) ** 2).sum((0, 2)))
    assert_parity(dg, out[sample], ref, TOL[prec], vol=vol, l2_scale=l2, elem_scale=(0.25 * R).abs().amax((0, 2)),
                  label=f"{size} p={p} {prec} stage")
    assert torch.isfinite(out).all()


@pytest.mark.parametrize("flux", ["rusanov", "roe"])
@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_vjp_of_disjoint_copies(p, prec, flux):
    """The adjoint of eight disjoint copies of a mesh (above the line) is eight times that of one
    (below it, the form the oracle tests run), to the rounding of another summation order."""
    mesh, _, U, W, _, _ = walls("below", p, "roe" if p % 2 else "rusanov")
    n_vert = int(mesh.elem_vid.max()) + 1

    def vjp(copies):
        shift = np.arange(copies)[:, None, None] * n_vert
        many = kuhn_cube(1, periodic=(False, False, True))
        many.elem_vid = (mesh.elem_vid[None] + shift).reshape(-1, 4)
        many.elem_xyz = np.tile(mesh.elem_xyz, (copies, 1, 1))
        many.bface_vid = (mesh.bface_vid[None] + shift).reshape(-1, 3)
        many.bface_tag = np.tile(mesh.bface_tag, copies)
        s = solver(p, prec, many, farfield=FAR)
        s.set_flux(flux)
        Ui, Wi, Yi = (s.set_state(X.repeat(copies, 1, 1).cuda()) for X in (U, W, U + W))
        return s.get_state(s.residual_vjp_axpy(Ui, Wi, 0.3, [(0.7, Yi)], s.new_state())).cpu().view(copies, *U.shape)

    one, eight = vjp(1), vjp(8)
    err = ((eight - one).norm() / (math.sqrt(8) * one.norm())).item()
    print(f"{prec} p={p} {flux}: copies differ by {err:.1e}")
    assert err < {"fp64": 1e-13, "fp32": 1e-5}[prec]
