"""The adjoint's transforms at every kind of grid (GPU): the vector-Jacobian product
of the density against the FP64 oracle.

Gathers of three inputs (the force chain) and nine (2LPT) run side by side in one
workgroup where grid and threads allow (sides up to 64), else one after the
other: at 8 both are wide, at 64 the nine inputs are wide in FP64 and not in
FP32, at 128 neither is.

Tolerances: those of the model tests, 1e-9 in FP64 and 1e-4 in FP32.  In FP32 a
particle whose position rounds to the other side of a cell face takes the
derivative of another cell, an error of the order of its own cotangent.  Positions
are off by 2e-6 cells at most (the 2LPT bound of the stage tests, 5e-6, on
displacements of 0.4 cells), two force evaluations and the data paint
read three coordinates each, so about 9 n^3 2e-6 particles do that; each
adds at most 4 / n^3 of the squared norm (twice its share)."""
import math

import numpy as np
import pytest

from gpu_common import cfg_small, context, model, rel_l2, require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu


def tolerance(n, prec):
    if prec == "f64":
        return 1e-9
    mean = 9 * n ** 3 * 2e-6
    crossings = math.floor(mean + 3 * math.sqrt(mean))
    return 1e-4 + math.sqrt(4.0 * crossings / n ** 3)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,nm", [(8, 8), (8, 16), (16, 32), (64, 64), (64, 128)])
def test_vjp_of_every_side(prec, n, nm):
    require_gpu()
    cfg = cfg_small(1, n_part=n, n_mesh=nm, n_steps=1, rsd="z", box=8.0 * n)
    ctx, mdl = context(cfg, prec), model(cfg)
    rng = np.random.default_rng(41)
    s, w = rng.standard_normal((2, n, n, n)).astype(np.float32).astype(np.float64)
    got = to_np(ctx.vjp(to_dev(s, prec), to_dev(w, prec)))
    err = rel_l2(got, mdl.vjp(s, w))
    print("vjp %d/%d %s: %.3e" % (n, nm, prec, err))
    assert err <= tolerance(n, prec)
