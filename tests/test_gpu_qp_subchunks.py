"""Quasi-periodic models: the smoother's sub-chunks (their number and length
follow from the chunk and the number of chunks) at lengths that end inside the
first sub-chunk, one step past a chunk and inside the last sub-chunk of a
chunk, with a zero step and long missing runs, against the oracle."""
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


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("J", [1, 2, 3])
@pytest.mark.parametrize("chunk,n", [(256, 1), (256, 17), (256, 257), (256, 1000), (40, 479), (16, 1601), (4, 90),
                                     (1000, 999)])
def test_subchunks(chunk, n, J, dtype):
    w = workloads.co2_like(max(n, 2), J=J, missing=0.2, seed_extra=n)
    t, y, mask = (w[k][:n] for k in ("t", "y", "mask"))
    t = t * (n / 1000.0 / t[-1]) * 30.0 if n > 1 else t  # 30 steps per unit of time and a few periods
    if n > 20:
        t[11] = t[10]
        mask[n // 2:n // 2 + n // 5] = 0
    yo = y if dtype == "float64" else y.astype(np.float32).astype(np.float64)
    c = w["model"]["components"]
    model = P.make_model(c, 0.01)
    r = P.predict(model, t, y, mask, dtype=dtype, options=P.make_options(chunk=chunk))
    ll = P.loglik(model, t, y, mask, dtype=dtype, options=P.make_options(chunk=chunk))
    o = oracle.run(OracleModel(c, 0.01), t, yo, mask)
    e = rel(r["f_mean"].double().cpu().numpy(), o["f_mean"]), rel(r["f_var"].double().cpu().numpy(), o["f_var"])
    print(J, dtype, chunk, n, "%.1e %.1e" % e, flush=True)
    assert P.status(r["ws"]) == 0
    assert e[0] <= TOL[dtype]["mean"] and e[1] <= TOL[dtype]["var"]
    assert float(r["loglik"]) == float(ll)
