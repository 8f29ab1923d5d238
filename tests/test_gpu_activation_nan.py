"""Layers without an activation hand on what their sums are, NaN and infinities included; rectified layers hand on zero for NaN."""
import numpy as np
import pytest

from helpers import gpu_run
from workloads import conv, maxpool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["none", "relu"])
@pytest.mark.parametrize("c_in,c_out,pool", [(3, 16, False), (16, 32, False), (32, 64, True)])
def test_sums_that_are_not_finite(act, c_in, c_out, pool):
    rng = np.random.default_rng(c_in)
    x = rng.normal(size=(2, 6, 20, c_in)).astype(np.float32)
    x[0, 2, 3, 1], x[0, 3, 12, 0], x[1, 4, 6, 2] = np.nan, np.inf, -np.inf
    w = rng.normal(0, 0.2, size=(c_out, c_in, 3, 3)).astype(np.float32)
    layers = [conv(c_in, c_out, 3, 3, p_h=1, p_w=1, act=act)] + ([maxpool(c_out)] if pool else [])
    wl = dict(name="nan", precision="f32", in_h=6, in_w=20, in_c=c_in, layers=layers, weights=[w] + [None] * pool, biases=[None] * len(layers),
              x=x, seg_rows=1, streams=2)
    got = gpu_run(wl, seg_rows=2)
    xp = np.pad(x.astype(np.float64), ((0, 0), (1, 1), (1, 1), (0, 0)))
    with np.errstate(invalid="ignore"):
        c = sum(np.einsum("byxc,oc->byxo", xp[:, ky:ky + 6, kx:kx + 20], w[:, :, ky, kx].astype(np.float64)) for ky in range(3) for kx in range(3))
    want = c if act == "none" else np.where(c > 0, c, 0.0)            # (NaN > 0 is false)
    if pool:
        # a NaN may win or lose against its neighbours in a window: windows without one are compared
        win = want.reshape(2, 3, 2, 10, 2, c_out)
        known = ~np.isnan(win).any(axis=(2, 4))
        want = np.where(known, np.nan_to_num(win, nan=-1.0, posinf=np.inf, neginf=-np.inf).max(axis=(2, 4)), 0.0)
        got = np.where(known, got, 0.0)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    ok = np.isfinite(want)
    assert np.array_equal(np.sign(got[~ok & ~np.isnan(want)]), np.sign(want[~ok & ~np.isnan(want)]))
    assert np.max(np.abs(got[ok] - want[ok])) <= 1e-4 * np.max(np.abs(want[ok]))
