"""Host-side checks of rules and arithmetic in the library's headers (CPU).

The functions that the kernels and their launch code share with the host are
compiled for the host alone (host_checks.hip) and called through ctypes."""
import ctypes
import os
import subprocess
from fractions import Fraction

import numpy as np
import pytest

from paper_2604_26823_amd import build

STATE = -7  # IC_ERR_STATE
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host") / "host_checks.so")
    cmd = [build.hipcc(), "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-fPIC",
           "-ffp-contract=off", "-shared", os.path.join(HERE, "host_checks.hip"), "-o", so]
    done = subprocess.run(cmd, capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
    lib = ctypes.CDLL(so)
    d, q = ctypes.c_double, ctypes.c_longlong
    lib.hc_unit.restype, lib.hc_unit.argtypes = d, [d]
    lib.hc_rounded.restype, lib.hc_rounded.argtypes = q, [d, d, d]
    lib.hc_particle.restype = None
    lib.hc_particle.argtypes = [ctypes.c_float, d, d, ctypes.POINTER(q)]
    lib.hc_gather_wide.argtypes = [ctypes.c_uint, ctypes.c_int, ctypes.c_int, q]
    lib.hc_sort_passes.argtypes = [ctypes.c_int, q]
    return lib


def contributions():
    """(amax, w, v): weights in [0, 1], products of three FP32 factors, |v| <= amax."""
    rng = np.random.default_rng(40)
    t = rng.random((400, 3), dtype=np.float32)
    w = (t[:, 0] * t[:, 1] * t[:, 2]).astype(np.float64)
    v = rng.standard_normal(400).astype(np.float32).astype(np.float64)
    out = []
    for amax in (1.0, float(np.abs(v).max()), 2.0 ** -140, np.nextafter(2.0, 1.0)):
        f = amax / np.abs(v).max()
        out += [(amax, a, float(b)) for a, b in zip(w, np.clip(v * f, -amax, amax))]
        out += [(amax, a, b) for a in (0.0, 0.5, 2.0 ** -51, 1.0 - 2.0 ** -24, 1.0)
                for b in (-amax, amax, 0.0, -amax * 2.0 ** -30)]
    return out


def test_fixed_point_contributions_round_to_2_52_of_the_largest(host):
    """A contribution w v of a work item whose largest |v| is amax: the integer is
    w v in units of the scale rounded to nearest, so off by at most half a unit,
    and the unit is at most 2^-51 amax (amax 2^e in [2^51, 2^52))."""
    for amax, w, v in contributions():
        unit = Fraction(host.hc_unit(amax))
        assert Fraction(amax) / unit < 2 ** 52
        assert unit <= Fraction(amax) / 2 ** 51
        got = host.hc_rounded(amax, w, v) * unit
        assert abs(got - Fraction(w) * Fraction(v)) <= unit / 2, (amax, w, v)


def particle(host, d, v, amax=1.0):
    out = (ctypes.c_longlong * 8)()
    host.hc_particle(d, v, amax, out)
    return list(out)


def test_particles_without_a_position_or_value_add_nothing(host):
    """A NaN or infinite displacement, and a NaN or infinite value, add nothing to the
    FP32 windows: their bit patterns are no integers."""
    whole = particle(host, 0.5, 1.0)
    assert sum(whole) == 2 ** 51 and min(whole) > 0
    nan, inf = float("nan"), float("inf")
    for d in (nan, inf, -inf):
        assert particle(host, d, 1.0) == [0] * 8, d
    for v in (nan, inf, -inf):
        assert particle(host, 0.5, v) == [0] * 8, v


def test_a_sort_of_one_value_is_one_pass(host):
    for size in (4, 8):
        assert host.hc_sort_passes(size, 1) == 1
        for n in (2, 1000, 1 << 20, 1 << 27):
            assert host.hc_sort_passes(size, n) == size


def test_scatter_outputs_must_not_share_storage(host):
    """On small grids each output of an x scatter is a workgroup row of its own that reads
    the inputs again: an output in an input's place, or in another output's, is refused."""
    assert host.hc_x_scatter(2, 3) == 0
    for o0, o1 in ((0, 3), (2, 1), (2, 2)):
        assert host.hc_x_scatter(o0, o1) == STATE, (o0, o1)


@pytest.mark.parametrize("n,prec,blocks,threads,lds,m,wide", [
    (8, "f32", 2, 64, 8 * 8 * 65, 9, 1), (16, "f64", 4, 64, 16 * 16 * 65, 9, 1),
    (32, "f64", 96, 32, 16 * 32 * 9, 9, 1), (64, "f32", 192, 128, 8 * 64 * 17, 3, 1),
    (64, "f64", 320, 64, 16 * 64 * 9, 3, 1), (64, "f32", 192, 128, 8 * 64 * 17, 9, 0),
    (64, "f64", 320, 64, 16 * 64 * 9, 9, 0), (64, "f64", 320, 64, 16 * 64 * 9, 1, 0),
    (128, "f32", 640, 256, 8 * 128 * 17, 3, 0), (128, "f64", 1152, 128, 16 * 128 * 9, 3, 0)])
def test_gathers_go_wide_where_all_their_workgroups_run_at_once(host, n, prec, blocks, threads,
                                                                lds, m, wide):
    """Side by side the inputs of a gather take m times the LDS and threads: only while
    the chip's 256 CUs hold every workgroup at once (nine inputs at 64^3 in FP64 fill
    a CU's LDS with one workgroup each, 320 of them)."""
    assert host.hc_gather_wide(blocks, m, threads, lds) == wide
