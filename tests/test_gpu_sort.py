"""The radix sort at the edges of its tiles (GPU): one element, wavefront and
tile boundaries of both tile shapes, the switch between them and between the
two ways of adding the chunk totals, with ties and signed zeros, subnormals
and a single digit throughout (all values equal), against the oracle's stable
descending order.  Orders are integers: equal, not close."""
import numpy as np
import pytest

from gpu_common import DEV, cfg_small, context, dt, require_gpu, torch
from oracle import rom

pytestmark = pytest.mark.gpu

SMALL_MAX = 1 << 20
SIZES = [1, 2, 63, 64, 65, 1023, 1024, 1025, 2047, 33 * 1024 + 1, 524_288, 524_289,
         SMALL_MAX - 1, SMALL_MAX, SMALL_MAX + 1, SMALL_MAX + 8191, 2_097_152, 2_097_153,
         4_194_305]


def _values(n, prec, kind):
    rng = np.random.default_rng(n)
    v = rng.standard_normal(n)
    if kind == "ties":
        v = np.round(v, 1)
        v[::3] = 0.0
        v[1::5] = -0.0
    elif kind == "equal":
        v[:] = 1.5
    elif kind == "tiny":
        v = v * np.finfo(np.float32).tiny * 1e-3  # subnormal in FP32
    return torch.tensor(v, dtype=dt(prec), device=DEV)


@pytest.mark.parametrize("kind", ["normal", "ties", "equal", "tiny"])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_sort_at_tile_edges(prec, kind):
    require_gpu()
    ctx = context(cfg_small(3, n_steps=1, lbfgs_m=1, tape_forces=0, nbar=1.0), prec)
    for n in SIZES:
        x = _values(n, prec, kind)
        got = ctx.sort_desc(x).cpu().numpy()
        assert np.array_equal(got, rom.descending_order(x.double().cpu().numpy())), (n, prec, kind)
