"""Sums over the tiles (log-likelihood, gradient) on either side of the number
of tiles up to which the last tile to finish forms them, against the same
calls at another number of steps per lane (FP64, 1e-10: sums of 16 384 terms
in another order and through other tiles), several calls on one workspace."""
import pytest

import workloads
from oracle.model import MATERN32
from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

import torch  # noqa: E402

import paper_2102_09964_amd as P  # noqa: E402


@pytest.mark.parametrize("n", [256, 257, 64 * 256, 64 * 256 + 1, 65 * 256 + 1])
def test_tile_sums(n):
    w = workloads.random_series(n, [(MATERN32, 0, 0.5, 1.0)], 0.01, span=0.05 * n, missing=0.2, seed=4)
    m = P.make_model([(MATERN32, 0, 0.5, 1.0)], 0.01)
    t, y = torch.as_tensor(w["t"], device="cuda"), torch.as_tensor(w["y"], device="cuda")
    mask = torch.as_tensor(w["mask"], device="cuda")
    out = []
    for chunk in (4, 33):
        o = P.make_options(chunk=chunk)
        pipe = P.Pipeline(m, n, "float64", options=o)
        ws = P.alloc_workspace(m, n, P.F64, P.OP_LOGLIK_GRAD, o)
        for _ in range(2):
            ll, g = P.loglik_grad(m, t, y, mask, dtype="float64", options=o, ws=ws)
            out.append((ll, g, pipe.run(t, y, mask)[2].item(), P.loglik(m, t, y, mask, dtype="float64", options=o)))
    ref = out[-1]
    for ll, g, l2, l3 in out:
        for a in (ll, l2, l3):
            assert abs(float(a) - float(ref[0])) <= 1e-10 * abs(float(ref[0]))
        d = torch.as_tensor(g) - torch.as_tensor(ref[1])
        assert d.norm() <= 1e-10 * torch.as_tensor(ref[1]).norm()
