"""Fused calls whose outputs overlap their inputs: all of an input is read before
the first output is written, so that smoothing the last result with the same
pipeline (its f_mean as observations), or writing the outputs over the times,
gives what separate buffers give. Sizes of more tiles than run at once, where a
tile could otherwise find its neighbour's output in place of an observation."""
import numpy as np
import pytest

import workloads
from oracle.model import MATERN32, RBF
from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

import torch  # noqa: E402

import paper_2102_09964_amd as P  # noqa: E402

MODELS = {"m32": [(MATERN32, 0, 0.5, 1.0)], "rbf4": [(RBF, 4, 1.0, 1.0)], "rbf6": [(RBF, 6, 1.0, 1.0)],
          "m32+rbf6": [(MATERN32, 0, 2.0, 0.5), (RBF, 6, 0.5, 0.5)]}


def _inputs(n, dtype):
    g = torch.Generator().manual_seed(n)
    t = torch.cumsum(torch.rand(n, generator=g, dtype=torch.float64), 0) * 0.02
    y = torch.sin(t) + 0.1 * torch.randn(n, generator=g, dtype=torch.float64)
    mask = (torch.rand(n, generator=g) >= 0.2).to(torch.uint8)
    return t.cuda(), y.to(getattr(torch, dtype)).cuda(), mask.cuda()


def check_overlaps(make, t, y, mask):
    """make() gives a pipeline; each overlap against separate buffers, bit for bit."""
    n = y.shape[0]
    want = [x.clone() for x in make().run(t.clone(), y.clone(), mask.clone())]
    for over in ("y=f_mean", "y=f_var", "t"):
        pipe, tt, yy = make(), t.clone(), y.clone()
        if over == "t":  # outputs over the times
            flat = tt.view(y.dtype)
            pipe.f_mean, pipe.f_var = flat[:n], (flat[n:2 * n] if flat.shape[0] >= 2 * n else pipe.f_var)
        else:
            yy = pipe.f_mean if over == "y=f_mean" else pipe.f_var
            yy.copy_(y)
        got = pipe.run(tt, yy, mask.clone())
        for a, b in zip(got, want):
            assert torch.equal(a, b), over


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("name", list(MODELS))
def test_single_series(name, dtype):
    n = 64 * 4 * 5000 + 3
    t, y, mask = _inputs(n, dtype)
    m = P.make_model(MODELS[name], 0.01)
    check_overlaps(lambda: P.Pipeline(m, n, dtype, options=P.make_options(chunk=4)), t, y, mask)


@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_batched(dtype):
    w = workloads.batched_matern(n_series=300, min_len=500, max_len=9000, missing=0.1, seed_extra=3)
    t, y, mask = (torch.as_tensor(w[k], device="cuda") for k in ("t", "y", "mask"))
    check_overlaps(lambda: P.BatchedPipeline(w["kinds"], w["offsets"], w["params"], dtype=dtype,
                                             options=P.make_options(chunk=4)),
                   t, torch.nan_to_num(y).to(getattr(torch, dtype)), mask.to(torch.uint8))


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("chunk", [16, 100])
def test_quasiperiodic(chunk, dtype):
    n = 100 * 2100 + 7
    t, y, mask = _inputs(n, dtype)
    m = P.make_model(workloads.co2_like(2, J=1)["model"]["components"], 0.01)
    check_overlaps(lambda: P.Pipeline(m, n, dtype, options=P.make_options(chunk=chunk)), t, y, mask)
