"""Training at the crop sizes where a weight gradient's workgroups take more
than one tile each and the input gradients form all output channels at once.

A layer's weight gradient runs min(tiles, 512 / block rows) workgroups that go
over the 4 x 4 x 16 tiles in turn: at crop 64 (1,024 tiles on the first level,
128 on the second) the two 16-channel layers and the 80 -> 32 one stage several
tiles, at crop 72 (1,620 tiles, 243 on the second level, the last of each row
partial, and beyond the node grid) with counts that do not divide.  Bars: those
of the gradient test on small crops (test_gpu_unet.py).

A context that only applies the network holds no training workspace.
"""
import numpy as np
import pytest

from oracle import unet

from ._pairs import Pair
from .test_gpu_unet import RHO_M, RHO_P, _blob, _dev, _pack, _params, _rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    from paper_2107_05123_amd import Context
    pair = Pair("uniform", 3, 6, 6)
    rng = np.random.default_rng(12)
    n = pair.lib.n_nodes
    phi, r, e = pair.phi("bubble", cn=0.02), rng.standard_normal(n), 3.0 * rng.standard_normal(n)
    params, K = _params(4), 2.5
    ctx = Context(pair.lib, Cn=0.02, rho_plus=RHO_P, rho_minus=RHO_M)
    ctx.pc_load(_blob(params, K))
    return pair, ctx, phi, r, e, params, K


@pytest.mark.parametrize("crop", [64, 72])
def test_gradients_over_several_tiles_match_oracle(setup, crop):
    pair, ctx, phi, r, e, params, K = setup
    loss = ctx.pc_train_step([_dev(phi)], [_dev(r)], [_dev(e)], [(0, 0, 0)], crop, flips=[3], lr=0.0)
    g = ctx.pc_gradients()
    X, T, mask = _pack(64, phi, r, e, (0, 0, 0), 3, crop, K)
    out, cache = unet.forward(params, X, store="bf16")
    L, dout = unet.mse(out, T, mask)
    assert abs(loss - L) <= 2e-2 * L, (loss, L)
    ref = unet.backward(cache, dout, store="bf16")
    off = 0
    for k, (ci, co) in enumerate(unet.layer_shapes()):
        gk = g[off:off + 27 * ci * co].reshape(27, ci, co).astype(np.float64)
        off += 27 * ci * co
        rk = ref["W"][k]
        if k == 0:
            gk, rk = gk[:, :2], rk[:, :2]
        print(f"crop {crop} layer {k}: {_rel(gk, rk):.2e}", flush=True)
        assert _rel(gk, rk) <= 5e-2, k
    assert _rel(g[off:].astype(np.float64), ref["w_out"]) <= 2e-2


def test_inference_holds_no_training_workspace(setup):
    from paper_2107_05123_amd import Context
    pair, _, phi, r, e, params, K = setup
    ctx = Context(pair.lib, Cn=0.02, rho_plus=RHO_P, rho_minus=RHO_M)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx.pc_load(_blob(params, K))
    held = free - torch.cuda.mem_get_info()[0]
    # weights, two moments and gradients in FP32 and the weights twice in bf16,
    # each allocation rounded up to 2 MiB at most, two small ones
    n = sum(27 * ci * co for ci, co in unet.layer_shapes())
    print(f"held {held / 2 ** 20:.1f} MiB of parameters {20 * n / 2 ** 20:.1f}", flush=True)
    assert held <= 20 * n + 8 * 2 ** 21
    # a first training step after that is the same as on a fresh context
    loss = [c.pc_train_step([_dev(phi)], [_dev(r)], [_dev(e)], [(0, 0, 0)], 16, lr=0.0) for c in (ctx, setup[1])]
    assert loss[0] == loss[1] and np.array_equal(ctx.pc_gradients(), setup[1].pc_gradients())
