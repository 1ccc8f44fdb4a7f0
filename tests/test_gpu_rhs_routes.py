"""Right-hand sides on every route their launch takes.

Octrees: the same forms on one octree cut into bricks of at most 8, 4, 2 and 1
leaves per edge.  At levels 5-8 the 4^3 bricks have more than 1,024 waves and
run in a kernel of their own beside the launch of the smaller classes; bricks
of 2 and 1 run in that launch alone, single leaves in an LDS kernel of their
own.  Levels 3-5 have few 4^3 bricks, merged with the others.  Every cut gives
the sums in another order only: 1e-12 relative (2-norm and max-norm).

Uniform 2D meshes against the oracle at the sides where the route or the chunk
length changes: 8^2 and 32^2 leaves (bricks), 64^2 (one row a wave; the brick
tests hold it too), 256^2 (two rows a wave, the last chunk shorter) and 512^2
(five rows, nine tiles).
"""
import numpy as np
import pytest

import chns_inputs as ci

from .test_gpu_bricks import (Case, _bubble_params, _close, _dev,
                              test_right_hand_sides_and_energy_match_oracle)  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (id, kind, dim, lmin, lmax, radius, band, Cn, brick classes)
CASES = [(f"uniform2d_l{lev}", "uniform", 2, lev, lev, 0.15, 0.03, cn, ())
         for lev, cn in ((3, 0.1), (5, 0.04), (6, 0.02), (8, 0.01), (9, 0.01))]


@pytest.fixture(scope="module", params=CASES, ids=lambda c: c[0])
def case(request):
    return Case(request.param)


@pytest.mark.parametrize("lmin,lmax,own4", [(3, 5, False), (5, 8, True)])
def test_brick_cuts_of_an_octree_agree(lmin, lmax, own4):
    from paper_2107_05123_amd import Context, Mesh, _lib as L
    ref = None
    for edge in (8, 4, 2, 1):
        mesh = Mesh(dim=3, min_level=lmin, max_level=lmax, rule="sphere_band", centres=[(0.5, 0.3, 0.5)],
                    radii=[0.15], band=0.0375, brick_max=edge)
        info = mesh.summary()
        print(f"edge {edge}: n={info['n_nodes']} hanging={info['n_hanging']} bricks={info['n_bricks']}", flush=True)
        assert info["n_hanging"] > 0
        if edge == 4:  # four 4^3 bricks to a wave
            assert (info["n_bricks"][1] > 4 * 1024) == own4
        if edge == 1:
            assert info["n_bricks"][:3] == [0, 0, 0]
        xyz = mesh.node_coords()
        order = np.lexsort(xyz.T)
        x = ci.unit_coords(xyz, lmax)
        wave = [np.cos(k * np.pi * x).prod(axis=1) for k in (1, 2, 3)]
        phi = ci.phi_bubble(x, cn=0.0125) + 0.02 * wave[2]
        u, v = np.concatenate(wave), np.concatenate(wave[::-1])
        base = [_dev(phi), _dev(0.1 * wave[0] * wave[1]), _dev(u), _dev(0.3 * v), _dev(wave[1])]
        ctx = Context(mesh, **_bubble_params(0.0125))
        got = [ctx.assemble(L.FORM_VP_RHS, base), ctx.assemble(L.FORM_PP_RHS, base + [_dev(v)]),
               ctx.assemble(L.FORM_VU_RHS, base + [_dev(v), _dev(wave[0])])]
        got = [g.cpu().numpy().reshape(-1, mesh.n_nodes)[:, order] for g in got]
        if ref is None:
            ref = got
        for a, b in zip(got, ref):
            _close(a, b)
