"""GPU parity of the one-kernel applies on uniform meshes at the edges of
their tiles: 3D FP64 pressure tiles complete 16 x 14 node columns, 2D waves 63
node columns, both in chunks of node layers or rows, so the sizes below are
one leaf or two per edge, just more than one tile, and several tiles and
chunks.  Every form, at the bars of the brick tests (the same checks run on
these meshes: 1e-12 relative, FP32 2e-5 of the largest entry).

The pressure coefficient takes four reciprocals from one at density ratios up
to 1e50 and one by one beyond; both are held to 1e-12 with a phase field that
stays away from the light phase (whose density the oracle's rho = alpha phi +
beta cannot hold at such ratios).
"""
import numpy as np
import pytest

from oracle import fem

from ._pairs import Pair
from .test_gpu_bricks import (Case, _close, _dev,  # noqa: F401
                              test_ch_residual_jacobian_and_diagonal_match_oracle,
                              test_momentum_apply_diagonal_and_scalar_operator_match_oracle,
                              test_pressure_apply_diagonal_and_rho_mass_match_oracle,
                              test_right_hand_sides_and_energy_match_oracle)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (id, kind, dim, lmin, lmax, radius, band, Cn, brick classes)
CASES = [("uniform3d_l1", "uniform", 3, 1, 1, 0.15, 0.03, 0.2, ()),
         ("uniform3d_l5", "uniform", 3, 5, 5, 0.15, 0.03, 0.04, ()),
         ("uniform2d_l1", "uniform", 2, 1, 1, 0.15, 0.03, 0.2, ()),
         ("uniform2d_l7", "uniform", 2, 7, 7, 0.15, 0.03, 0.02, ())]


@pytest.fixture(scope="module", params=CASES, ids=lambda c: c[0])
def case(request):
    return Case(request.param)


@pytest.mark.parametrize("ratio", [1e-3, 1e-45, 1e-55, 1e55])
def test_joint_and_single_reciprocals_match_oracle(ratio):
    from paper_2107_05123_amd import Context
    pair = Pair("uniform", 3, 3, 3)
    rng = np.random.default_rng(2)
    phi = rng.uniform(-0.5, 1.5, pair.lib.n_nodes) * (1.0 if ratio < 1 else -1.0)
    ctx = Context(pair.lib, rho_plus=1.0, rho_minus=ratio)
    ctx.set_phase_field(_dev(phi))
    A = fem.pp_matrix(pair.orc, pair.to_orc(phi), 1.0, ratio)
    x = rng.standard_normal(pair.lib.n_nodes)
    _close(ctx.apply(ctx.PRESSURE, _dev(x)).cpu().numpy(), pair.to_lib(A @ pair.to_orc(x)))


@pytest.mark.parametrize("dim,level", [(3, 5), (2, 7)])
def test_fused_sweeps_and_dots_solve_to_tolerance(dim, level):
    """The damped-Jacobi sweep and the p.Ap sum inside the apply: multigrid
    and Jacobi CG reach 1e-8, measured with the oracle's matrix."""
    from paper_2107_05123_amd import Context
    pair = Pair("uniform", dim, level, level)
    phi = pair.phi("bubble", cn=0.04)
    ctx = Context(pair.lib, rho_plus=1.0, rho_minus=1e-3)
    ctx.set_phase_field(_dev(phi))
    A = fem.pp_matrix(pair.orc, pair.to_orc(phi), 1.0, 1e-3)
    b = np.random.default_rng(4).standard_normal(pair.lib.n_nodes)
    b -= b.mean()
    for pc in ("gmg", "jacobi"):
        x, st = ctx.solve_pressure(_dev(b), pc=pc)
        bo = pair.to_orc(b)
        res = np.linalg.norm(bo - A @ pair.to_orc(x.cpu().numpy())) / np.linalg.norm(bo)
        print(pc, st, res, flush=True)
        assert res <= 1.05e-8
