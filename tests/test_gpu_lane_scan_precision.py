"""Precision of the lane scan in a launch of its own (d >= 6): filter moments of
a dense series at small noise against a sequential filter in extended precision
on the library's own transitions, the library's bars (tests.parity.TOL) on the
posterior, and the two forms of the FP32 scan (up to 512 tiles and beyond),
which do the same operations, bit for bit."""
import numpy as np
import pytest

import workloads
from oracle.model import MATERN32, RBF
from tests.conftest import gpu_available
from tests.parity import TOL, rel

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

import torch  # noqa: E402

import paper_2102_09964_amd as P  # noqa: E402

MODELS = {"rbf6": [(RBF, 6, 1.0, 1.0)], "m32+rbf6": [(MATERN32, 0, 2.0, 0.5), (RBF, 6, 0.5, 0.5)]}


def _sequential(m, t, y, noise):
    """h m and h P h^T of the filter, one step after the other in extended precision."""
    H = P.model_matrices(m)[2].astype(np.longdouble)
    d = len(H)
    F, Q = P.discretize(m, t)
    F = F.cpu().numpy().astype(np.longdouble)
    Q = P.unpack_sym(Q, d).cpu().numpy().astype(np.longdouble)
    mm, PP = np.zeros(d, np.longdouble), np.zeros((d, d), np.longdouble)
    out = np.empty((2, len(t)))
    for k in range(len(t)):
        mp, Pp = F[k] @ mm, F[k] @ PP @ F[k].T + Q[k]
        Ph = Pp @ H
        K = Ph / (H @ Ph + noise)
        mm, PP = mp + K * (y[k] - H @ mp), Pp - np.outer(K, Ph)
        out[:, k] = H @ mm, H @ PP @ H
    return out


@pytest.mark.parametrize("chunk", [64])
@pytest.mark.parametrize("name", list(MODELS))
def test_filter_moments_fp64(name, chunk):
    """Gaps of a thousandth of a unit, noise variance 1e-6. Rounding the prediction
    of a prior of size 1 to FP64 puts 1e-16 into a filtered variance of a tenth of
    the noise, 1e-9 of it; a hundred times that for the steps that it lasts. (64
    steps a lane: the rounding of the aggregates of 16 steps each alone puts 3e-6
    there for the sum, whatever the scan does.)"""
    rng = np.random.default_rng(21)
    n, noise = 1100, 1e-6
    t = np.cumsum(1e-3 * rng.exponential(size=n))
    y = np.sin(2 * t) + 1e-3 * rng.normal(size=n)
    m = P.make_model(MODELS[name], noise)
    H = torch.as_tensor(P.model_matrices(m)[2], device="cuda")
    o = P.filter(m, t, y, dtype="float64", options=P.make_options(chunk=chunk))
    Pf = P.unpack_sym(o["P"], len(H))
    r = _sequential(m, t, y, noise)
    e = rel((H @ o["m"]).cpu().numpy(), r[0]), rel((Pf @ H @ H).cpu().numpy(), r[1])
    print(name, chunk, "%.1e %.1e" % e, flush=True)
    assert e[0] <= 1e-7 and e[1] <= 1e-7


@pytest.mark.parametrize("name", list(MODELS))
@pytest.mark.parametrize("n", [257, 3 * 256 + 9, 512 * 256 + 1])
def test_bars(name, n):
    w = workloads.random_series(n, MODELS[name], 0.01, span=0.02 * n, missing=0.3, seed=n % 89)
    w["mask"][n // 3:n // 2] = 0
    m, o = P.make_model(MODELS[name], 0.01), P.make_options(chunk=4)
    t, y = torch.as_tensor(w["t"], device="cuda"), torch.as_tensor(w["y"], device="cuda")
    mask = torch.as_tensor(w["mask"], device="cuda")
    r = P.plain_predict(m, t, y, mask)
    for dtype in ("float64", "float32"):
        a = P.predict(m, t, y.to(getattr(torch, dtype)), mask, dtype=dtype, options=o)
        for k, b in (("f_mean", "mean"), ("f_var", "var")):
            e = rel(a[k].double().cpu().numpy(), r[k].cpu().numpy())
            print(name, n, dtype, k, "%.1e" % e, flush=True)
            assert e <= TOL[dtype][b], (dtype, k)
    # (FP32: of the log-likelihood of the same FP32-rounded observations)
    r32 = P.loglik(m, t, y.float().double(), mask, dtype="float64", options=o)
    for x, ref, dtype in ((P.loglik(m, t, y, mask, dtype="float64", options=o), r["loglik"], "float64"),
                          (a["loglik"], r32, "float32")):
        x, ref = (float(v["loglik"] if isinstance(v, dict) else v) for v in (x, ref))
        print(name, n, dtype, "loglik %.1e" % (abs(x - ref) / abs(ref)), flush=True)
        assert abs(x - ref) <= TOL[dtype]["loglik"] * abs(ref)


def test_fp32_forms_agree_bitwise():
    """d = 8: the moments of a step depend on the steps before it alone, so those of
    512 tiles are the same in a call of 512 tiles (the scan in its own launch) and
    of 513 (in the fold)."""
    n = 512 * 256
    w = workloads.random_series(n + 1, MODELS["m32+rbf6"], 0.01, span=0.02 * n, missing=0.3, seed=5)
    m, o = P.make_model(MODELS["m32+rbf6"], 0.01), P.make_options(chunk=4)
    a = P.filter(m, w["t"][:n], w["y"][:n], w["mask"][:n], dtype="float32", options=o)
    b = P.filter(m, w["t"], w["y"], w["mask"], dtype="float32", options=o)
    for k in ("m", "P"):
        assert torch.equal(a[k], b[k][:, :n].contiguous()), k
