"""Quasi-periodic models at observation noise far below the signal, as
test_gpu_small_noise.py for the one-lane scans: the library's bars
(tests.parity.TOL) against the oracle."""
import numpy as np
import pytest

import oracle
import workloads
from oracle.model import OracleModel
from tests.conftest import gpu_available
from tests.parity import TOL, rel

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

import torch  # noqa: E402

import paper_2102_09964_amd as P  # noqa: E402


def _check(J, gap, noise, missing, dtype, chunk, n=700):
    rng = np.random.default_rng(31)
    c = workloads.co2_like(2, J=J)["model"]["components"]
    t = np.cumsum(gap * (0.5 + rng.random(n)))
    y = np.sin(2 * np.pi * t) + 0.5 * np.sin(t / 30.0) + np.sqrt(noise) * rng.normal(size=n)
    y = y.astype(np.float32).astype(np.float64)
    mask = (rng.random(n) >= missing).astype(np.uint8)
    if missing:
        mask[n // 4:n // 3] = 0
    r = P.predict(P.make_model(c, noise), t, y, mask, dtype=dtype, options=P.make_options(chunk=chunk))
    o = oracle.run(OracleModel(c, noise), t, y, mask)
    e = rel(r["f_mean"].double().cpu().numpy(), o["f_mean"]), rel(r["f_var"].double().cpu().numpy(), o["f_var"])
    print(J, gap, noise, dtype, chunk, "%.1e %.1e" % e, "status", P.status(r["ws"]), flush=True)
    assert P.status(r["ws"]) == 0
    assert e[0] <= TOL[dtype]["mean"] and e[1] <= TOL[dtype]["var"]


@pytest.mark.parametrize("chunk", [16, 64])
@pytest.mark.parametrize("noise", [1e-4, 1e-10, 1e-14])
@pytest.mark.parametrize("J", [1, 2, 3])
def test_between_observations(J, noise, chunk):
    """FP64, gaps of a tenth of the longest length-scale, a third of the steps test
    points."""
    _check(J, 5.0, noise, 0.3, "float64", chunk)


@pytest.mark.parametrize("chunk", [16, 64])
@pytest.mark.parametrize("noise", [1e-2, 1e-10, 1e-18])
@pytest.mark.parametrize("J", [1, 2, 3])
def test_between_observations_fp32(J, noise, chunk):
    """As above in FP32, whose chunks' moments differ by their rounding, and, at the
    smallest noise, a filtered variance of f below the rounding of the predicted
    one."""
    _check(J, 5.0, noise, 0.3, "float32", chunk)


@pytest.mark.parametrize("chunk", [16, 64])
@pytest.mark.parametrize("J,gap,noise", [(J, 5.0, r) for J in (1, 2, 3) for r in (1e-2, 1e-3)] + [(2, 1.0, 1e-4)])
def test_every_step_observed_fp32(J, gap, noise, chunk):
    """Every step observed, f_var of the size of the noise. (At 1e-4 the rounding of
    the chunks' FP32 moments puts 6e-5 to 1.0e-4 into f_var whatever the smoother
    does; 12 states stay clear of the bar.)"""
    _check(J, gap, noise, 0.0, "float32", chunk)

