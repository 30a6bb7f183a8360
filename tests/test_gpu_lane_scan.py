"""Lane scan in a launch of its own (d >= 6) against the plain scan: tiles with
one lane, all lanes and one step more, several tiles, missing stretches that
leave identity-like aggregates, and either side of the number of tiles up to
which FP32 takes it. FP64: 1e-8 of the plain scan (the bar of the fused
smoother's tests). FP32: the log-likelihood of a chunk does not depend on how
many tiles follow, so it is compared with FP64 at the FP32 bar."""
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


@pytest.mark.parametrize("name", list(MODELS))
@pytest.mark.parametrize("n", [1, 4, 5, 255, 256, 257, 3 * 256 + 9, 512 * 256, 512 * 256 + 1])
def test_lane_scan(name, n):
    w = workloads.random_series(n, MODELS[name], 0.01, span=0.02 * n, missing=0.3, seed=n % 89)
    w["mask"][n // 3:n // 2] = 0
    m, o = P.make_model(MODELS[name], 0.01), P.make_options(chunk=4)
    t, y = torch.as_tensor(w["t"], device="cuda"), torch.as_tensor(w["y"], device="cuda")
    mask = torch.as_tensor(w["mask"], device="cuda")
    r = P.plain_predict(m, t, y, mask)
    a = P.predict(m, t, y, mask, dtype="float64", options=o)
    b = P.predict(m, t, y.float(), mask, dtype="float32", options=o)
    for k in ("f_mean", "f_var"):
        assert rel(a[k].cpu().numpy(), r[k].cpu().numpy()) <= 1e-8, k
        assert rel(b[k].double().cpu().numpy(), r[k].cpu().numpy()) <= TOL["float32"]["mean" if k == "f_mean" else "var"], k
    for x, tol in ((a, 1e-8), (b, 1e-4)):
        assert abs(float(x["loglik"]) - float(r["loglik"])) <= tol * max(1.0, abs(float(r["loglik"])))
