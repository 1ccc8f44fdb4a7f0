"""GPU parity of the one-pass diagonals of the scalar operators on octrees
with hanging nodes in every arrangement: random refinement (each octant split
with probability 0.35 by a hash of its place and level), so that leaves meet
coarser ones across faces, edges and both at once, in 2D and 3D, besides a
band mesh and a carved column.  Bar: 1e-12 relative (2-norm and max-norm)
against the diagonal of the oracle's assembled matrix, every operator.
"""
import random

import numpy as np
import pytest

import chns_inputs as ci
from oracle import chns, fem, mesh as om

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (id, dim, lmin, lmax, hash seed (None: slab), carve level, extent)
MESHES = [("random3d_a", 3, 1, 4, 1, 0, (0, 0, 0)), ("random3d_b", 3, 2, 5, 2, 0, (0, 0, 0)),
          ("random2d_a", 2, 1, 5, 3, 0, (0, 0, 0)), ("random2d_b", 2, 2, 6, 4, 0, (0, 0, 0)),
          ("column3d", 3, 3, 5, None, 3, (2, 8, 1))]


@pytest.mark.parametrize("spec", MESHES, ids=lambda m: m[0])
def test_one_pass_diagonals_match_oracle(spec):
    from paper_2107_05123_amd import Context, Mesh
    name, dim, lmin, lmax, seed, carve, extent = spec
    side = 1 << lmax

    def split(anchor, level):
        if seed is None:
            return ci.rt_slab_meets(anchor[1] / side, (anchor[1] + (side >> level)) / side, 1.0)
        return random.Random(repr((seed, level, tuple(int(a) for a in anchor[:dim])))).random() < 0.35

    def pred(level, lo, hi):
        return split([round(v * side) for v in lo] + [0] * (3 - dim), level)
    lib = Mesh(dim=dim, min_level=lmin, max_level=lmax, rule="callback", refine=split, carve_level=carve,
               extent=extent)
    box = [e / (1 << carve) for e in extent[:dim]] if carve else None
    orc = om.from_predicate(dim, lmin, lmax, pred, box)
    perm = om.node_index_map(lib.node_coords(), orc.indep_coords(), side)
    info = lib.summary()
    print(f"{name}: n={info['n_nodes']} hanging={info['n_hanging']} bricks={info['n_bricks']}", flush=True)
    assert info["n_hanging"] > 0
    prm_kw = dict(Re=35.0, We=10.0, Cn=0.05, Fr=1.0, rho_plus=1.0, rho_minus=1e-3, eta_plus=1.0, eta_minus=1e-2,
                  dt=5e-4)
    prm = chns.Params(**prm_kw)
    ctx = Context(lib, **prm_kw)
    phi_o = np.random.default_rng(7).uniform(-1.3, 1.3, lib.n_nodes)
    ctx.set_phase_field(torch.tensor(phi_o[perm], device="cuda"))
    qp = fem.qp_values(orc, phi_o)
    el = chns.Elems(orc)
    zero = np.zeros((dim, lib.n_nodes))
    state = chns.QPState(el, prm, phi_o, zero[0], zero, zero, zero[0])
    scalar = fem.mass_matrix(orc, prm.rho(qp)) / prm.dt + fem.stiffness_matrix(orc, prm.eta(qp)) / (2 * prm.Re)
    for op, mat in ((ctx.PRESSURE, fem.pp_matrix(orc, phi_o, 1.0, 1e-3)), (ctx.MASS, fem.mass_matrix(orc)),
                    (ctx.MOMENTUM_SCALAR, scalar), (ctx.MASS_RHO, chns.rho_mass_walls(el, prm, state))):
        got = ctx.diagonal(op).cpu().numpy().reshape(-1, lib.n_nodes)
        ref = mat.diagonal()[perm]
        for d in got:
            assert np.linalg.norm(d - ref) <= 1e-12 * np.linalg.norm(ref), op
            assert np.abs(d - ref).max() <= 1e-12 * np.abs(ref).max(), op
