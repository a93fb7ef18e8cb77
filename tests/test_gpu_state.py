"""The calls around a run, for every order and state type: layout round trip, volume points,
projection and admissibility count, on a ragged mesh and on one that a wavefront of the persistent
kernels takes several groups of."""
import numpy as np
import pytest
import torch

from synthetic import fields, kuhn_cube

pytestmark = pytest.mark.gpu

from gpu_common import solver  # noqa: E402
from paper_2209_01877_amd import debug_tables  # noqa: E402


@pytest.mark.parametrize("n", [(5, 4, 3), (23, 22, 23)])  # 360 and 69,828 elements
@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_calls_around_a_run(p, prec, n):
    mesh = kuhn_cube(n, length=1.0, jitter=0.2, shuffle_seed=2209, vid_seed=2210)
    s = solver(p, prec, mesh)
    E, NP, NQ = mesh.n_elem, s.n_modes, s.n_vol_points
    xi, w, B = (torch.from_numpy(debug_tables(p, k).reshape(shape))
                for k, shape in ((0, (NQ, 3)), (1, (NQ,)), (4, (NQ, NP))))
    # layout round trip: exact
    U = torch.from_numpy(fields.random_coefficients(E, NP, seed=3, scale=0.01))
    if prec == "fp32":
        U = U.float().double()
    Ui = s.set_state(U.cuda())
    assert torch.equal(s.get_state(Ui).cpu(), U)
    assert not Ui[:, -1, :, NP - 4 * (-(-NP // 4) - 1):].any()  # the last quad's unused modes
    # volume points: one affine map, a few roundings of coordinates of size 1
    X = torch.from_numpy(np.take_along_axis(mesh.elem_xyz, np.argsort(mesh.elem_vid, 1)[:, :, None], 1))
    x = X[:, :1] + xi @ (X[:, 1:] - X[:, :1])
    assert (s.volume_points().cpu() - x).abs().max() < 16 * 2.0 ** -53
    # projection: N_q products, relative to the largest coefficient
    q = fields.RandomSmooth(5)(x)
    rho, u, pr = q[..., :1], q[..., 1:4], q[..., 4:]
    cons = torch.cat([rho, rho * u, pr / 0.4 + 0.5 * rho * (u * u).sum(-1, keepdim=True)], -1)
    ref = 6.0 * cons.transpose(1, 2) @ (w[:, None] * B)
    err = (s.get_state(s.project(q.cuda())).cpu() - ref).abs().max() / ref.abs().max()
    assert err < (2.0 ** -23 if prec == "fp32" else 2 * NQ * 2.0 ** -53)
    # admissibility: the first, the last and a few other elements of the internal order
    assert int(s.check_state(Ui)) == 0
    bad = [0, E - 1, E // 2, E // 3]
    for k, b in enumerate(bad):
        e = int(s.perm[b])
        if k % 2:
            U[e, 4, 0] = -1.0
        else:
            U[e, 1 + k // 2, NP - 1] = float("nan")
    assert int(s.check_state(s.set_state(U.cuda()))) == len(bad)
