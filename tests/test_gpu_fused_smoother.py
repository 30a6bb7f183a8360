"""The fused call's smoother (lane ends joined by the scan, the Bryson-Frazier
recursion inside a lane) where its differences cancel most and where lanes and tiles end: small noise against the predicted variance,
long gaps of missing steps, series starts inside lanes, one step more or less
than a tile. FP32 and the batched form against the oracle; FP64 single series
against the library's plain scan of the same elements, because at this noise
the RBF model's stationary covariance (its Lyapunov residual of 1e-11) alone
puts both 5e-10 to 1.3e-9 from the oracle."""
import numpy as np
import pytest

import oracle
import workloads
from oracle.model import MATERN12, MATERN32, MATERN52, RBF, OracleModel
from tests.conftest import gpu_available
from tests.parity import TOL, rel

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

import torch  # noqa: E402

import paper_2102_09964_amd as P  # noqa: E402

MODELS = {"m12": [(MATERN12, 0, 0.5, 1.0)], "m32": [(MATERN32, 0, 0.5, 1.0)], "m52": [(MATERN52, 0, 1.0, 1.0)],
          "rbf6": [(RBF, 6, 1.0, 1.0)], "m32+rbf6": [(MATERN32, 0, 2.0, 0.5), (RBF, 6, 0.5, 0.5)]}


@pytest.mark.parametrize("dtype,chunk", [("float64", 1), ("float64", 5), ("float64", 64), ("float32", 4), ("float32", 16)])
@pytest.mark.parametrize("name", list(MODELS))
def test_edges(name, dtype, chunk):
    # the FP32 bars hold at the noise of the workloads (0.01); FP64 is also
    # held at a hundredth of it
    noise = 1e-4 if dtype == "float64" else 1e-2
    for n in (1, 2, 64 * chunk - 1, 64 * chunk, 64 * chunk + 1, 3 * 64 * chunk + 7):
        w = workloads.random_series(n, MODELS[name], noise, span=0.05 * n, missing=0.5, gap="exponential", seed=n % 97)
        w["mask"][n // 3:n // 2] = 0  # a long gap
        pipe = P.Pipeline(P.make_model(MODELS[name], noise), n, dtype, options=P.make_options(chunk=chunk))
        fm, fv, _ = pipe.run(torch.as_tensor(w["t"], device="cuda"),
                             torch.as_tensor(w["y"], device="cuda", dtype=getattr(torch, dtype)),
                             torch.as_tensor(w["mask"], device="cuda"))
        if dtype == "float64":
            r = P.plain_predict(P.make_model(MODELS[name], noise), w["t"], w["y"], w["mask"])
            o = {k: r[k].cpu().numpy() for k in ("f_mean", "f_var")}
        else:
            o = oracle.run(OracleModel(MODELS[name], noise), w["t"], w["y"].astype(np.float32).astype(np.float64),
                           w["mask"])
        e = rel(fm.double().cpu().numpy(), o["f_mean"]), rel(fv.double().cpu().numpy(), o["f_var"])
        print(name, dtype, chunk, n, "%.1e %.1e" % e, flush=True)
        assert P.status(pipe.ws_p) == 0
        assert e[0] <= TOL[dtype]["mean"] and e[1] <= TOL[dtype]["var"]


@pytest.mark.parametrize("chunk", [1, 7, 64])
def test_series_starts_inside_lanes(chunk):
    """FP64, noise variances down to 1e-6: at a series start S / R is 1e6,
    digits that the rank-one update must not lose."""
    w = workloads.batched_matern(n_series=40, min_len=1, max_len=200, missing=0.3, seed_extra=21)
    w["params"][:, 2] = np.exp(np.linspace(np.log(1e-6), np.log(1e-2), 40))
    pipe = P.BatchedPipeline(w["kinds"], w["offsets"], w["params"], dtype="float64", options=P.make_options(chunk=chunk))
    fm, fv, _ = pipe.run(torch.as_tensor(w["t"], device="cuda"), torch.as_tensor(w["y"], device="cuda"),
                         torch.as_tensor(w["mask"], device="cuda"))
    models = [OracleModel([(int(k), 0, float(p[0]), 1.0)], float(p[2])) for k, p in zip(w["kinds"], w["params"])]
    o = oracle.run_batched(models, w["offsets"], w["t"], w["y"], w["mask"], threads=4)
    worst = [0.0, 0.0]
    for a, b in zip(w["offsets"][:-1], w["offsets"][1:]):
        worst[0] = max(worst[0], rel(fm[a:b].cpu().numpy(), o["f_mean"][a:b]))
        worst[1] = max(worst[1], rel(fv[a:b].cpu().numpy(), o["f_var"][a:b]))
    print(chunk, worst, flush=True)
    assert max(worst) <= 1e-9
