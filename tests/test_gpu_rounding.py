"""Rounding of the folded constants.

The light phase is held exactly: with phi = -1 everywhere every mixture
coefficient is the light phase's, so an apply is the equal-density one times
rho- (the pressure operator: over rho-).  At density and viscosity ratios of
1e-8 a coefficient formed as a difference of two rounded halves is off by 1e-8;
the bar is 1e-13 of the largest entry (a few roundings of 64 bits in sums of up
to 32 leaf contributions).

FP32 constants do not bias a result: the Cahn-Hilliard Jacobian in FP32 on
inputs and parameters that FP32 holds exactly, its projection on the FP64 apply
of the same inputs within 2e-8 of one.  The roundings of the arithmetic are
independent from leaf to leaf and average out (5e-8 over the root of 10^4
entries); what is left is the transforms' own constant (six transforms of 1e-9,
the square of the phase field as many again).  One constant rounded to FP32 is
up to 6e-8.
"""
import numpy as np
import pytest

from ._pairs import Pair

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MESHES = [("uniform", 2, 5, 5), ("band", 2, 3, 6), ("uniform", 3, 4, 4), ("band", 3, 2, 4)]


def _dev(a, dt=torch.float64):
    return torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")


@pytest.mark.parametrize("mesh", MESHES, ids=lambda m: f"{m[0]}{m[1]}d")
def test_light_phase_coefficients_are_exact(mesh):
    from paper_2107_05123_amd import Context
    pair = Pair(*mesh, band=0.1)
    n, ratio = pair.lib.n_nodes, 1e-8
    rng = np.random.default_rng(3)
    xyz = pair.lib.node_coords()
    wall = ((xyz == 0) | (xyz == 1 << mesh[3])).any(axis=1)
    kw = dict(Re=35.0, We=10.0, Cn=0.05, dt=5e-4, rho_plus=1.0, eta_plus=1.0)
    ctx = Context(pair.lib, rho_minus=ratio, eta_minus=ratio, **kw)
    one = Context(pair.lib, rho_minus=1.0, eta_minus=1.0, **kw)
    for c in (ctx, one):
        c.set_phase_field(_dev(np.full(n, -1.0)))
        c.set_coefficients(c.MOMENTUM, [_dev(np.full(n, -1.0)), _dev(np.zeros(n)), _dev(np.zeros(mesh[1] * n))])
    for name, factor in (("PRESSURE", 1.0 / ratio), ("MASS_RHO", ratio), ("MOMENTUM_SCALAR", ratio),
                         ("MOMENTUM", ratio)):
        op = getattr(ctx, name)
        x = rng.standard_normal((ctx.fields(op), n))
        if name in ("MASS_RHO", "MOMENTUM"):
            x[:, wall] = 0.0  # identity rows
        got, ref = (c.apply(op, _dev(x.reshape(-1))).cpu().numpy() for c in (ctx, one))
        err = np.abs(got / factor - ref).max() / np.abs(ref).max()
        print(f"{mesh} {name}: {err:.1e}", flush=True)
        assert err <= 1e-13, name
        if name != "MOMENTUM":
            got, ref = (c.diagonal(op).cpu().numpy().reshape(-1, n)[:, ~wall] for c in (ctx, one))
            assert np.abs(got / factor - ref).max() <= 1e-13 * np.abs(ref).max(), name


@pytest.mark.parametrize("mesh", [("uniform", 2, 7, 7), ("uniform", 3, 5, 5), ("band", 3, 3, 6)],
                         ids=lambda m: f"{m[0]}{m[1]}d")
def test_fp32_jacobian_is_not_biased(mesh):
    from paper_2107_05123_amd import Context
    pair = Pair(*mesh, band=0.1)
    n, dim = pair.lib.n_nodes, mesh[1]
    rng = np.random.default_rng(4)
    ctx = Context(pair.lib, Re=32.0, We=8.0, Cn=2.0 ** -7, Pe=2.0 ** 20, rho_plus=1.0, rho_minus=2.0 ** -10,
                  eta_plus=1.0, eta_minus=2.0 ** -6, dt=0.5)

    def field(k, scale):  # multiples of 2^-12
        return _dev(np.round(scale * rng.standard_normal(k) * 4096) / 4096)
    phi = field(n, 0.5)
    ctx.set_coefficients(ctx.CH_JACOBIAN, [phi, phi, field(dim * n, 0.25)])
    x = field(2 * n, 1.0)
    y64 = ctx.apply(ctx.CH_JACOBIAN, x).reshape(2, n)
    y32 = ctx.apply(ctx.CH_JACOBIAN, x.float()).double().reshape(2, n)
    for k in range(2):
        bias = float((y32[k] @ y64[k]) / (y64[k] @ y64[k]) - 1)
        print(f"{mesh} row {k}: {bias:.1e}", flush=True)
        assert abs(bias) <= 2e-8, k
