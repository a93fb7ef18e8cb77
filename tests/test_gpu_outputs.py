"""What the calls write into outputs that hold garbage (NaN) before, and of infinite inputs."""
import pytest
import torch

from synthetic import fields

pytestmark = pytest.mark.gpu

from gpu_common import make_mesh, oracle, random_state, solver  # noqa: E402
from paper_2209_01877_amd import debug_tables  # noqa: E402


def unused_modes(s, X):
    r = s.n_modes % 4
    return X[:, -1, :s.n_elem, r:] if r else X[:, -1, :s.n_elem, 4:]


def garbage(s):
    return torch.full(s.state_shape, float("nan"), dtype=s.state_dtype, device="cuda")


@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_viscous_padding_is_written_as_zeros(p, prec):
    """Elements past the mesh: a caller may reduce over the padded array of a residual or stage."""
    mesh = make_mesh("ragged")
    s = solver(p, prec, mesh, mu=0.02)
    U = s.set_state(random_state(oracle(p, mesh), seed=71).cuda())
    for out in (s.residual(U, garbage(s)), s.rk_stage(U, U, garbage(s), 0.75, 1e-3)):
        s.sync()
        assert torch.isfinite(out[:, :, :s.n_elem]).all()
        assert not out[:, :, s.n_elem:].any()
        assert not unused_modes(s, out).any()


@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16", "fp16"])
def test_states_and_residuals_are_written_whole(p, prec):
    mesh = make_mesh("ragged")
    s = solver(p, prec, mesh)
    user = random_state(oracle(p, mesh), seed=72).cuda()
    U = s.set_state(user, garbage(s))
    x = s.volume_points()
    P = s.project(fields.RandomSmooth(5)(x).contiguous(), garbage(s))
    R = s.residual(U, garbage(s))
    S = s.rk_stage(U, U, garbage(s), 0.75, 1e-3)
    s.sync()
    for X in (U, P, R, S):
        assert torch.isfinite(X[:, :, :s.n_elem]).all()
        assert not unused_modes(s, X).any()
    # set_state and project fill the padding with a copy of the first element
    for X in (U, P):
        assert torch.equal(X[:, :, s.n_elem:], X[:, :, :1].expand_as(X[:, :, s.n_elem:]))


@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_projection_of_an_infinite_point(p, prec):
    """An infinite pressure at one point makes every energy coefficient infinite, with the sign of
    the mode at that point; the last point of the rule is where a padded contraction would
    multiply it by a zero weight."""
    mesh = make_mesh("ragged")
    s = solver(p, prec, mesh)
    NQ, NP = s.n_vol_points, s.n_modes
    B = torch.from_numpy(debug_tables(p, 4).reshape(NQ, NP))
    prim = torch.ones(mesh.n_elem, NQ, 5, dtype=torch.float64)
    points = {3: NQ - 1, 5: 0}
    for e, q in points.items():
        prim[e, q, 4] = float("inf")
    got = s.get_state(s.project(prim.cuda())).cpu()
    s.sync()
    for e, q in points.items():
        assert (B[q] != 0).all()
        assert torch.equal(got[e, 4], torch.sign(B[q]) * float("inf")), (q, got[e, 4])
        assert torch.isfinite(got[e, :4]).all()
    got[list(points), 4] = 0.0
    assert torch.isfinite(got).all()
