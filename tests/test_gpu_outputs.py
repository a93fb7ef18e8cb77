"""What the calls write into outputs that hold garbage (NaN) before."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from gpu_common import make_mesh, oracle, random_state, solver  # noqa: E402


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
