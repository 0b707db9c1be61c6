"""Small contributions beside large ones in an FP32 paint (GPU).

The windows of an FP32 paint sum in fixed point with a unit of 2^-51 of the
largest contribution (1 in a density paint), so each contribution is rounded by
at most 2^-52."""
import numpy as np
import pytest

from gpu_common import cfg_small, context, require_gpu, to_dev, to_np

pytestmark = pytest.mark.gpu

N, CELL, UNIT = 8, 8.0, 2.0 ** -51


@pytest.mark.parametrize("grid", [0, 1])
@pytest.mark.parametrize("units", [1.0, 1.5, 5.0])
def test_a_contribution_of_one_unit_is_kept(grid, units):
    """Particle 0 lies units x 2^-51 of a cell above its lattice point, all others on
    the cell (4, 4, 4), all in one work item."""
    require_gpu()
    ctx = context(cfg_small(1, n_part=N, n_mesh=N, n_steps=1, rsd="z", box=CELL * N), "f32")
    q = np.stack(np.meshgrid(*[np.arange(N)] * 3, indexing="ij")).reshape(3, -1)
    d = (4.0 - q) * CELL
    d[:, 0] = [units * UNIT * CELL, 0.0, 0.0]
    rho = to_np(ctx.paint(to_dev(d, "f32"), grid))
    assert abs(rho[1, 0, 0] - units * UNIT) <= UNIT / 2
    assert rho[0, 0, 0] == 1.0 and rho[4, 4, 4] == N ** 3 - 1
