"""The kernels' branches by grid side, axis and particle distribution (GPU),
against the FP64 oracle on the same inputs.

Which kernel runs depends on the side and the precision: whole planes (n <=
128, and 256 in FP32) or separate y and z passes; x passes that split a
workgroup by output or input on small grids; one-launch orders up to 4096
blocks; wavefront tiles of the lattice down to 8^3; halos added by the FFT or,
at 256 in FP32, partly before it.

Tolerances.  Transforms: those of the stage tests (an FFT accumulates a few
units of rounding per axis; the multipliers weigh error and field alike).
Forces: those of the stage test.  Paints of clustered particles: a cell is the
sum of at most `items` work items' own sums and seven halo values, each rounded to
the working precision, so its error is at most (items + 16) units of rounding
(16 for the weights' own, three products of values with one rounding each,
and the conversions) times the largest cell; in FP64 the oracle's positions
carry a rounding of the box coordinate besides, a unit per cell of the side, in
each of up to eight particles per unit of density (a corner's weight is an eighth
on average)."""
import numpy as np
import pytest

from gpu_common import (DEV, cfg_small, context, model, np_dt, rel_l2, require_gpu, to_dev,
                        to_np, torch)
from oracle import cic, fourier, upsample
from paper_2604_26823_amd import inputs
from paper_2604_26823_amd.api import Context

pytestmark = pytest.mark.gpu

PRECS = ["f32", "f64"]
EPS = {"f32": 2.0 ** -24, "f64": 2.0 ** -53}


def small(n, nm=None):
    return cfg_small(1, n_part=n, n_mesh=nm or n, n_steps=2, rsd="z", box=8.0 * n)


WHITE, GRAD, HESS = 1, 2, 4


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n", [8, 16, 64, 128])
@pytest.mark.parametrize("kinds,a,b", [(GRAD, 0, 0), (GRAD, 1, 0), (GRAD, 2, 0), (HESS, 0, 2),
                                       (HESS, 1, 1), (WHITE, 0, 0), (WHITE | GRAD, 1, 0),
                                       (GRAD | HESS, 0, 0), (GRAD | HESS, 2, 1)])
def test_multipliers_of_every_side_and_axis(prec, n, kinds, a, b):
    require_gpu()
    cfg = small(n)
    ctx, mdl = context(cfg, prec), model(cfg)
    x = np.random.default_rng(31).standard_normal((n, n, n)).astype(np_dt(prec)).astype(np.float64)
    m = np.ones((n, n, n // 2 + 1), dtype=np.complex128)
    if kinds & WHITE:
        m = m * mdl.mult("white")
    if kinds & GRAD:
        m = m * mdl.mult("grad", a)
    if kinds & HESS:
        m = m * mdl.mult("hess", (a, b))
    got = to_np(ctx.multiplier(to_dev(x, prec), kinds, a, b))
    assert rel_l2(got, fourier.apply(m, x)) <= (5e-6 if prec == "f32" else 1e-12)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n", [8, 16, 64, 128])
def test_lpt_of_every_side(prec, n):
    require_gpu()
    cfg = small(n)
    ctx, mdl = context(cfg, prec), model(cfg)
    s = np.random.default_rng(32).standard_normal((n, n, n)).astype(np.float32).astype(np.float64)
    d, p = ctx.lpt(to_dev(s, prec))
    d0, p0, _ = mdl.lpt(s)
    tol = 5e-6 if prec == "f32" else 1e-12
    assert rel_l2(to_np(d), d0) <= tol
    assert rel_l2(to_np(p), p0) <= tol


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n,nm", [(8, 8), (8, 16), (16, 16), (64, 128), (128, 128), (128, 256)])
def test_forces_of_every_side(prec, n, nm):
    require_gpu()
    cfg = small(n, nm)
    ctx, mdl = context(cfg, prec), model(cfg)
    d = np.random.default_rng(33).normal(0, 6.0, (3, n ** 3)).astype(np_dt(prec)).astype(np.float64)
    ref, _ = mdl.force(d)
    assert rel_l2(to_np(ctx.force(to_dev(d, prec))), ref) <= (2e-5 if prec == "f32" else 1e-11)


def clustered(mdl, n, box, keep):
    """Displacements that bring all but every keep-th particle into a sphere of a
    few cells across a corner shared by eight blocks (and the box face)."""
    rng = np.random.default_rng(34)
    target = rng.normal(0.0, 0.02 * box, (3, n ** 3))
    d = target - mdl.q
    d[:, ::keep] = rng.normal(0, 4.0, d[:, ::keep].shape)
    return d


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n,nm", [(16, 16), (32, 64)])
def test_blocks_of_many_items_and_empty_blocks(prec, n, nm):
    require_gpu()
    cfg = small(n, nm)
    ctx, mdl = context(cfg, prec), model(cfg)
    d = clustered(mdl, n, cfg["box"], 97).astype(np_dt(prec)).astype(np.float64)
    items = n ** 3 // 1024 + 1
    for grid, cells, cell in [(0, n, mdl.dq), (1, nm, mdl.dm)]:
        got = to_np(ctx.paint(to_dev(d, prec), grid))
        ref = cic.paint(mdl.q + d, cells, cell)
        bound = (items + 16 + (8 * cells if prec == "f64" else 0)) * EPS[prec] * ref.max()
        assert np.max(np.abs(got - ref)) <= bound
    ref, _ = mdl.force(d)
    assert rel_l2(to_np(ctx.force(to_dev(d, prec))), ref) <= (2e-5 if prec == "f32" else 1e-11)


@pytest.mark.parametrize("prec", PRECS)
def test_upsampling_from_the_smallest_grid(prec):
    require_gpu()
    cfg = lambda n: inputs.config(1, n_part=n, n_mesh=n, box=500.0, n_steps=1, tape_forces=0,
                                  lbfgs_m=1)
    s_low = inputs.white_noise(8, 108)
    ref = upsample.upsample(s_low.astype(np.float64), 16, cfg(16)["seed"], 5)
    low, high = Context(cfg(8), prec, DEV), Context(cfg(16), prec, DEV)
    try:
        got = to_np(high.upsample_from(low, torch.tensor(s_low, dtype=low.dtype, device=DEV), 5))
    finally:
        high.close()
        low.close()
    assert rel_l2(got, ref) <= (2e-6 if prec == "f32" else 1e-12)
