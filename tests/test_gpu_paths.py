"""Parity at the sizes where a kernel's split of the work changes: U-Net crops
of one partial tile, of fewer than 256 tiles on every level (each 16-channel
block in a workgroup of its own) and of 432 tiles on the first; 2D steps whose
Cahn-Hilliard and momentum systems (33,282 unknowns) run the small-system GMRES
kernels with a ragged last block, and (132,098) the general ones.
"""
import pytest

from oracle import unet

from .test_gpu_chns import Case, _compare_states, _oracle_steps, _run_steps
from .test_gpu_unet import _dev, _pack, _rel, setup  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("crop", [8, 40, 48])
def test_forward_over_tile_counts_matches_oracle(setup, crop):  # noqa: F811
    # the bar of the forward test of test_gpu_unet.py
    ctx, pair, phi, r, e, params, K = setup
    out = ctx.pc_forward(_dev(phi), _dev(r), origin=(0, 0, 0), flip=0, crop=crop).cpu().numpy()
    X, _, _ = _pack(16, phi, r, e, (0, 0, 0), 0, crop, K)
    ref, _ = unet.forward(params, X, store="bf16")
    assert _rel(out.reshape(crop, crop, crop), ref) <= 2e-2


@pytest.mark.parametrize("level", [7, 8])
def test_step_over_system_sizes_matches_oracle(level):
    # the bar of the step tests: the worst conditioned solve, the pressure's,
    # amplifies its residual of 1e-11 by at most (1 / h)^2 = 65,536
    c = Case(("uniform", 2, level, level, "drop2d", 0.02))
    state, _ = _run_steps(c, 1)
    st, _ = _oracle_steps(c, 1)
    _compare_states(c, state, st, 1e-6)
