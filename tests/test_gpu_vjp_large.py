"""The FP64 P3 adjoint above the line where groups are no longer split (10,752 groups of 16 elements on
256 CUs), and the FP64 P4 adjoint between 768 and 1,024 groups: disjoint copies of a mesh against one
copy, which the split form takes."""
import math

import numpy as np
import pytest
import torch

from synthetic import fields, kuhn_cube

pytestmark = pytest.mark.gpu

from gpu_common import solver  # noqa: E402

FAR = (1.0, 0.5 * math.sqrt(1.4), 0.0, 0.0, 1.0)


@pytest.mark.parametrize("p,copies", [(3, 47), (4, 4)])  # 11,104 and 948 groups
def test_copies(p, copies):
    mesh = kuhn_cube((10, 9, 7), periodic=(False, False, True), jitter=0.2, bump_height=0.05, shuffle_seed=2209,
                     vid_seed=2210)

    def vjp(n):
        shift = np.arange(n)[:, None, None] * (int(mesh.elem_vid.max()) + 1)
        many = kuhn_cube(1, periodic=(False, False, True))
        many.elem_vid = (mesh.elem_vid[None] + shift).reshape(-1, 4)
        many.elem_xyz = np.tile(mesh.elem_xyz, (n, 1, 1))
        many.bface_vid = (mesh.bface_vid[None] + shift).reshape(-1, 3)
        many.bface_tag = np.tile(mesh.bface_tag, n)
        s = solver(p, "fp64", many, farfield=FAR)
        U, W = (torch.from_numpy(fields.random_coefficients(mesh.n_elem, s.n_modes, seed=k, scale=0.01)).repeat(n, 1, 1)
                for k in (41, 42))
        Ui, Wi = s.set_state(U.cuda()), s.set_state(W.cuda())
        out = torch.full_like(Ui, float("nan"))
        return s.get_state(s.residual_vjp_axpy(Ui, Wi, 0.3, [(0.7, Wi)], out)).cpu().view(n, mesh.n_elem, 5, -1)

    one, many = vjp(1), vjp(copies)
    # sums of a few hundred fp64 products in another order
    assert (many - one).norm() < 1e-13 * math.sqrt(copies) * one.norm()
    assert (many - one).abs().max() < 1e-13 * one.abs().max()
