"""FP64 transition of the RBF blocks (Taylor series of degree 10, 13 or 16,
chosen per wave by its longest step, and squarings beyond): the FP64 filter
and smoother against the oracle over step lengths on both sides of every
switch (0.035, 0.076 and 0.2 length-scales at order 6), and the gradient."""
import numpy as np
import pytest

import oracle
import workloads
from oracle.model import MATERN32, RBF, OracleModel
from tests.conftest import gpu_available
from tests.parity import rel

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

import torch  # noqa: E402

import paper_2102_09964_amd as P  # noqa: E402

MODELS = {"rbf3": [(RBF, 3, 1.0, 1.0)], "rbf4": [(RBF, 4, 1.0, 1.0)], "rbf6": [(RBF, 6, 1.0, 1.0)],
          "m32+rbf6": [(MATERN32, 0, 2.0, 0.5), (RBF, 6, 0.5, 0.5)]}


@pytest.mark.parametrize("gap", [0.01, 0.05, 0.2, 1.0, 5.0])
@pytest.mark.parametrize("name", list(MODELS))
def test_step_lengths(name, gap):
    n = 700
    w = workloads.random_series(n, MODELS[name], 0.01, span=gap * n, gap="exponential", seed=11)
    w["t"][100] = w["t"][99]  # a zero step
    model = P.make_model(MODELS[name], 0.01)
    t = torch.as_tensor(w["t"], device="cuda")
    y = torch.as_tensor(w["y"], device="cuda")
    mask = torch.as_tensor(w["mask"], device="cuda")
    pipe = P.Pipeline(model, n, "float64", options=P.make_options(chunk=4))
    fm, fv, ll = pipe.run(t, y, mask)
    om = OracleModel(MODELS[name], 0.01, with_derivatives=True)
    o = oracle.run(om, w["t"], w["y"], w["mask"], gradient=True)
    e = [rel(fm.cpu().numpy(), o["f_mean"]), rel(fv.cpu().numpy(), o["f_var"]),
         abs(float(ll.cpu()[0]) - o["loglik"]) / abs(o["loglik"])]
    print(name, gap, ["%.1e" % v for v in e], flush=True)
    assert P.status(pipe.ws_p) == 0
    assert max(e) <= 1e-9
    _, g = P.loglik_grad(model, t, y, mask, dtype="float64", options=P.make_options(chunk=4))
    # the tests of the gradient hold FP64 to 1e-8 of the largest component
    assert rel(g.cpu().numpy(), o["grad"]) <= 1e-8
