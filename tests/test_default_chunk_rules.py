"""The default number of steps per lane or team (options.chunk = 0) is the rule that
the interface states, by state size and type: results are those of that chunk
given explicitly, bit for bit, either side of the lengths where it changes."""
import pytest

import paper_2102_09964_amd as P
import workloads
from oracle.model import MATERN32, RBF
from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

import torch  # noqa: E402


def _same(model, n, dtype, chunk):
    g = torch.Generator().manual_seed(n)
    t = (torch.cumsum(torch.rand(n, generator=g, dtype=torch.float64), 0) * 0.02).cuda()
    y = (torch.sin(t) + 0.1 * torch.randn(n, generator=g, dtype=torch.float64).cuda()).to(getattr(torch, dtype))
    m = P.make_model(model, 0.01)
    a = P.predict(m, t, y, dtype=dtype)
    b = P.predict(m, t, y, dtype=dtype, options=P.make_options(chunk=chunk))
    for k in ("f_mean", "f_var", "loglik"):
        assert torch.equal(a[k], b[k]), (k, n, chunk)
    assert P.status(a["ws"]) == 0


@pytest.mark.parametrize("n,chunk", [(1, 4), (257, 4), (131072, 4), (131073, 5), (262145, 9), (524288, 16), (524289, 9),
                                     (1048577, 16)])
def test_rbf6_fp64(n, chunk):
    """d = 6: 512 tiles a round of the lane scan, two rounds beyond 2^19 steps."""
    _same([(RBF, 6, 1.0, 1.0)], n, "float64", chunk)


@pytest.mark.parametrize("n,dtype,chunk", [(1, "float64", 8), (1000, "float64", 8), (131072, "float64", 8),
                                           (131073, "float64", 9), (262144, "float64", 16), (262145, "float64", 9),
                                           (786433, "float64", 16), (20011, "float32", 16)])
def test_sum_d8(n, dtype, chunk):
    """d = 8: from 8 steps a lane, whose scan rounds less than that of 4; 256 tiles a
    round."""
    _same([(MATERN32, 0, 2.0, 0.5), (RBF, 6, 0.5, 0.5)], n, dtype, chunk)


@pytest.mark.parametrize("J,n,dtype,chunk", [(1, 1000, "float64", 16), (1, 65537, "float64", 17), (1, 262107, "float64", 64),
                                             (2, 1000, "float64", 64), (3, 131073, "float64", 65), (1, 70001, "float32", 256)])
def test_quasiperiodic(J, n, dtype, chunk):
    _same(workloads.co2_like(2, J=J)["model"]["components"], n, dtype, chunk)
