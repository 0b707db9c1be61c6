"""What the library's timing report says about its launches (GPU)."""
import numpy as np
import pytest

from gpu_common import cfg_small, model, np_dt, require_gpu, to_dev, to_np
from oracle import cic
from paper_2604_26823_amd.api import Context

pytestmark = pytest.mark.gpu

PRECS = ["f32", "f64"]


def recorded(ctx, call):
    """The report's rows by kernel name of one call, and its result."""
    ctx.timing(True)
    out = call()
    rows = {r["name"]: r for r in ctx.timing_report()}
    ctx.timing(False)
    return rows, out


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("nm", [16, 32])
def test_deterministic_paint_takes_no_halo_pass(prec, nm):
    """A deterministic paint converts its integer sums to the complete field: no pass
    over a halo follows it (tolerance: that of the stage tests' paints)."""
    require_gpu()
    n = 16
    cfg = cfg_small(1, n_part=n, n_mesh=nm, n_steps=1, rsd="z", box=8.0 * n, deterministic=1)
    mdl = model(cfg_small(1, n_part=n, n_mesh=nm, n_steps=1, rsd="z", box=8.0 * n))
    d = np.random.default_rng(35).normal(0, 6.0, (3, n ** 3)).astype(np_dt(prec)).astype(float)
    ctx = Context(cfg, prec, "cuda:0")
    try:
        ctx.force(to_dev(d, prec))  # leaves a halo behind
        for grid, cells, cell in [(0, n, mdl.dq), (1, nm, mdl.dm)]:
            rows, rho = recorded(ctx, lambda: ctx.paint(to_dev(d, prec), grid))
            assert "cic_paint" in rows and "halo_add" not in rows
            ref = cic.paint(mdl.q + d, cells, cell)
            assert np.max(np.abs(to_np(rho) - ref)) <= (2e-5 if prec == "f32" else 1e-11)
    finally:
        ctx.close()


def spectrum_bytes(n, elem):
    return n * n * (n // 2 + 1) * 2 * elem


def halo_entries(n):
    """Entries of a paint's halo: three faces, three edges and a corner per 8^3
    block, rounded up to 32."""
    b = n // 8
    return (3 * n * n * b + 3 * n * b * b + b ** 3 + 31) // 32 * 32


@pytest.mark.parametrize("prec", PRECS)
def test_report_counts_the_fields_of_every_launch(prec):
    """bytes_per_launch of the fused inverse passes over launches of one field (the
    multiplier) and of six (2LPT, twice): the mean, each field read as a half
    spectrum and written once."""
    require_gpu()
    n, elem = 16, 4 if prec == "f32" else 8
    ctx = Context(cfg_small(1, n_part=n, n_mesh=n, n_steps=1, rsd="z", box=8.0 * n), prec, "cuda:0")
    try:
        x = to_dev(np.random.default_rng(36).standard_normal((n, n, n)), prec)
        rows, _ = recorded(ctx, lambda: (ctx.lpt(x), ctx.multiplier(x, 2)))
        row = rows["fft_c2r_yz"]
        field = n ** 3 * elem + spectrum_bytes(n, elem)
        assert row["count"] == 3
        assert abs(row["bytes"] - (6 + 6 + 1) * field / 3) <= 1e-6 * field
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("det", [0, 1])
def test_report_counts_what_a_paint_writes(prec, det):
    """A paint reads positions and ids and writes its field and halo, once each."""
    require_gpu()
    n, elem = 16, 4 if prec == "f32" else 8
    ctx = Context(cfg_small(1, n_part=n, n_mesh=n, n_steps=1, rsd="z", box=8.0 * n,
                            deterministic=det), prec, "cuda:0")
    try:
        d = to_dev(np.random.default_rng(37).normal(0, 6.0, (3, n ** 3)), prec)
        rows, _ = recorded(ctx, lambda: ctx.paint(d, 0))
        out = (n ** 3 + halo_entries(n)) * (8 if det else elem)
        assert rows["cic_paint"]["bytes"] == n ** 3 * (3 * elem + 4) + out
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", PRECS)
def test_report_counts_what_a_step_moves(prec):
    """The step of a one-step run reads positions, momenta (through the order's map) and
    ids, the force meshes once, and writes both states and one packed rank; the
    2LPT state is counted into its order by a key and a rank per particle."""
    require_gpu()
    n, elem = 16, 4 if prec == "f32" else 8
    ctx = Context(cfg_small(1, n_part=n, n_mesh=n, n_steps=1, rsd="z", box=8.0 * n), prec, "cuda:0")
    try:
        s = to_dev(np.random.default_rng(38).standard_normal((n, n, n)), prec)
        rows, _ = recorded(ctx, lambda: ctx.evolve(s))
        assert rows["pm_step"]["bytes"] == n ** 3 * (12 * elem + 12) + 3 * n ** 3 * elem
        assert rows["sort_keys"]["bytes"] == n ** 3 * (3 * elem + 8)
        d = to_dev(np.random.default_rng(39).normal(0, 6.0, (3, n ** 3)), prec)
        rows, _ = recorded(ctx, lambda: ctx.paint(d, 0))
        assert rows["sort_scatter"]["bytes"] == n ** 3 * (6 * elem + 16)
    finally:
        ctx.close()
