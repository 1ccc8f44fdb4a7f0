"""Two properties of the multigrid preconditioners that the smoother's kernels
carry: the V-cycle is a fixed symmetric linear map, and its convergence does
not depend on the mesh.

Symmetry.  One CG iteration from zero returns a multiple of M^-1 b, so the
products of M^-1 come out of the public solve up to a factor each: with b3 =
b1 + b2, x3 = c1 x1 + c2 x2 and c1 x1 and c2 x2 are M^-1 b1 and M^-1 b2 times
one number.  The fused sweep y = x + w D^-1 (r - A x) runs on one side of the
cycle against the zero-guess sweep and the unfused product on the other, so a
sweep that is wrong somewhere (a tile's rim, the weight) leaves b2.M^-1 b1 and
b1.M^-1 b2 apart.  Bar 1e-5 of the geometric mean of b1.M^-1 b1 and
b2.M^-1 b2: the coarse operators are rounded to FP32 entry by entry (27 entries
of 2^-24); a rim of one node in sixteen left out is 1e-2.

Mesh independence.  The Cahn-Hilliard Schur preconditioner smooths a shifted
pressure operator with its one-pass diagonal on octrees, with the probed one on
uniform meshes.  With a diagonal short of the shift the sweeps diverge; the
iterations of the same step on an octree and on the uniform mesh of its finest
level stay within half as many again.
"""
import numpy as np
import pytest

import chns_inputs as ci

from ._pairs import Pair

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("kind,dim,lmin,lmax", [("uniform", 3, 3, 3), ("uniform", 3, 5, 5), ("uniform", 3, 6, 6),
                                                ("uniform", 2, 5, 5), ("uniform", 2, 7, 7), ("band", 3, 3, 5)])
def test_vcycle_is_linear_and_symmetric(kind, dim, lmin, lmax):
    from paper_2107_05123_amd import Context, Mesh
    band = dict(rule="sphere_band", centres=[(0.5, 0.3, 0.5)[:dim]], radii=[0.15], band=0.06)
    mesh = Mesh(dim=dim, min_level=lmin, max_level=lmax, **(band if kind == "band" else dict(rule="uniform")))
    x = ci.unit_coords(mesh.node_coords(), lmax)
    ctx = Context(mesh, rho_plus=1.0, rho_minus=1e-3)
    ctx.set_phase_field(_dev(ci.phi_bubble(x, cn=0.04)))
    rng = np.random.default_rng(5)
    b = rng.standard_normal((2, mesh.n_nodes))
    b -= b.mean(axis=1, keepdims=True)
    b = np.concatenate([b, b.sum(axis=0, keepdims=True)])
    out = []
    for k in range(3):
        xk, st = ctx.solve_pressure(_dev(b[k]), pc="gmg", rtol=1e-14, max_it=1, raise_on_noconv=False)
        assert st.iterations == 1
        xk = xk.cpu().numpy()
        out.append(xk - xk.mean())
    c, *_ = np.linalg.lstsq(np.stack(out[:2], axis=1), out[2], rcond=None)
    z1, z2 = c[0] * out[0], c[1] * out[1]
    assert np.linalg.norm(z1 + z2 - out[2]) <= 1e-10 * np.linalg.norm(out[2])
    gap = abs(b[1] @ z1 - b[0] @ z2) / np.sqrt((b[0] @ z1) * (b[1] @ z2))
    print(f"{kind} {dim}D {lmin}-{lmax}: symmetry {gap:.1e}", flush=True)
    assert gap <= 1e-5


@pytest.mark.parametrize("dim,lmin,lmax", [(2, 4, 7), (3, 3, 5)])
def test_schur_iterations_on_an_octree_and_on_its_finest_mesh(dim, lmin, lmax):
    from paper_2107_05123_amd import Context
    its = []
    for kind in ("band", "uniform"):
        pair = Pair(kind, dim, lmin, lmax, band=0.08)
        ctx = Context(pair.lib, Re=35.0, We=10.0, Cn=0.04, rho_plus=1.0, rho_minus=1e-3, eta_plus=1.0,
                      eta_minus=1e-2, dt=5e-4)
        phi = _dev(pair.phi("bubble", cn=0.04))
        u = torch.zeros(dim * pair.lib.n_nodes, dtype=torch.float64, device="cuda")
        state = {"u": u, "u_prev": u.clone(), "p": torch.zeros_like(phi), "phi": phi, "mu": ctx.initial_mu(phi)}
        s = ctx.advance_step(state, ch_pc="schur", pp_pc="gmg", vp_pc="gmg")
        print(f"{kind} {dim}D {lmin}-{lmax}: newton {s['newton']} ch {s['ch_iterations']}", flush=True)
        its.append(s["ch_iterations"] / sum(s["newton"]))
    assert its[0] <= 1.5 * its[1] + 1
