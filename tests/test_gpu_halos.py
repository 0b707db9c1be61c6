"""Painted fields with halos at the sizes the small tests do not reach (GPU): dense
and empty blocks on a 256^3 mesh (orders above 4096 blocks; at 256 in FP32 the x
halo is added apart), and the 1024^3 mesh, whose forward z pass takes fewer rows
per workgroup than a block has.

Tolerances.  Paints of clustered particles: (items + 16) units of rounding of
the largest cell, `items` work items' own sums added to a cell, plus in FP64
the oracle's positions, a unit per cell of the side in each of eight particles
per unit of density.  Forces: 2e-5 in FP32 and 1e-11 in FP64 (those of the stage
tests), or the paint's own bound where that is larger."""
import numpy as np
import pytest

from gpu_common import (DEV, cfg_small, model, np_dt, rel_l2, require_gpu, to_dev, to_np, torch)
from oracle import cic
from paper_2604_26823_amd import _lib
from paper_2604_26823_amd.api import Context
from test_gpu_kernel_paths import EPS, clustered
from test_gpu_large import _mesh_context

pytestmark = pytest.mark.gpu

TOL_FORCE = {"f32": 2e-5, "f64": 1e-11}


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_clustered_particles_on_a_256_mesh(prec):
    require_gpu()
    n, nm = 128, 256
    cfg = cfg_small(1, n_part=n, n_mesh=nm, n_steps=1, rsd="z", box=8.0 * n)
    mdl = model(cfg)
    d = clustered(mdl, n, cfg["box"], 97).astype(np_dt(prec)).astype(np.float64)
    items = n ** 3 // 1024 + 1
    ctx = Context(cfg, prec, DEV)
    try:
        rho = to_np(ctx.paint(to_dev(d, prec), 1))
        F = to_np(ctx.force(to_dev(d, prec)))
    finally:
        ctx.close()
    ref = cic.paint(mdl.q + d, nm, mdl.dm)
    bound = (items + 16 + (8 * nm if prec == "f64" else 0)) * EPS[prec]
    assert np.max(np.abs(rho - ref)) <= bound * ref.max()
    assert rel_l2(F, mdl.force(d)[0]) <= max(TOL_FORCE[prec], bound)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_force_of_a_1024_mesh_adds_the_halo(prec):
    """The force chain reads a painted field and its halo apart; the same field painted
    complete, transformed, multiplied by i k_a / k^2 in torch, transformed back
    and read out at 2^18 particles gives the same force."""
    require_gpu()
    nm, n = 1024, 512
    ctx = _mesh_context(nm, prec)
    cell = 4.0
    try:
        gen = torch.Generator(device=DEV)
        gen.manual_seed(42)
        d = torch.empty(3, n ** 3, dtype=ctx.dtype, device=DEV)
        d.normal_(0.0, 6.0, generator=gen)
        sel = torch.randint(n ** 3, (1 << 18,), generator=gen, device=DEV)
        F = ctx.force(d)[:, sel].double()
        rho = ctx.paint(d, _lib.IC_GRID_MESH)
        rho -= n ** 3 / nm ** 3
        X = ctx.rfft(rho, grid=_lib.IC_GRID_MESH)
        del rho
        m = torch.arange(nm, device=DEV)
        k = torch.where(m < nm // 2, m, m - nm).double() * (2 * np.pi / (nm * cell))
        kd = torch.where(m == nm // 2, torch.zeros_like(k), k)  # derivative: 0 at Nyquist
        kz = k[:nm // 2 + 1].abs()
        axes = [kd[:, None, None], kd[None, :, None], kd[None, None, :nm // 2 + 1]]
        inv = k[:, None, None] ** 2 + k[None, :, None] ** 2 + kz[None, None, :] ** 2
        inv[0, 0, 0] = 1.0
        inv = (1.0 / inv).to(ctx.dtype)
        site = torch.stack([sel // (n * n), sel // n % n, sel % n])
        x = site * (nm // n) + d[:, sel].double() / cell  # in cells
        del d
        base = torch.floor(x)
        t = x - base
        base = base.long()
        ref = torch.zeros(3, sel.numel(), dtype=torch.float64, device=DEV)
        for a in range(3):
            f = (axes[a] * (nm ** 3 / n ** 3)).to(ctx.dtype) * inv
            G = torch.complex(-X.imag * f, X.real * f)
            del f
            g = ctx.irfft(G, grid=_lib.IC_GRID_MESH).view(-1)
            del G
            for corner in range(8):
                o = [corner >> 2 & 1, corner >> 1 & 1, corner & 1]
                w = torch.ones(sel.numel(), dtype=torch.float64, device=DEV)
                i = torch.zeros_like(sel)
                for q in range(3):
                    w *= t[q] if o[q] else 1.0 - t[q]
                    i = i * nm + (base[q] + o[q]) % nm
                ref[a] += w * g[i].double()
            del g
        err = rel_l2(to_np(F), to_np(ref))
        torch.cuda.synchronize()
    finally:
        ctx.close()
        del ctx
        torch.cuda.empty_cache()
    print("1024^3 force %s: %.3e" % (prec, err))
    assert err <= TOL_FORCE[prec]
