"""The default number of steps per lane (options.chunk = 0) of the FP64 scans
grows with the series, from 4 to 16 steps (FP32: 16): the workspace of a longer series serves every
shorter one, the static scratch takes what it took with 16 steps, and the
results are those of the same chunk given explicitly."""
import numpy as np
import pytest

import paper_2102_09964_amd as P
from oracle.model import MATERN32, RBF
from tests.conftest import gpu_available

MODELS = {"m32": [(MATERN32, 0, 0.5, 1.0)], "rbf6": [(RBF, 6, 1.0, 1.0)],
          "m32+rbf6": [(MATERN32, 0, 2.0, 0.5), (RBF, 6, 0.5, 0.5)]}


def _expected(n, lanes):
    return min(16, max(4, -(-n // lanes)))


@pytest.mark.parametrize("dtype", [P.F32, P.F64])
@pytest.mark.parametrize("name", list(MODELS))
def test_workspace_monotone_and_static_scratch(name, dtype):
    m = P.make_model(MODELS[name], 0.01)
    rng = np.random.default_rng(5)
    ns = set(int(v) for v in np.exp(rng.uniform(0, np.log(3e6), 400)))
    for lanes in (49152, 65536):
        ns |= {k * lanes + j for k in range(1, 18) for j in (-1, 0, 1)}
    ns = sorted(n for n in ns if n > 0)
    for op in (P.OP_FILTER, P.OP_SMOOTH, P.OP_LOGLIK, P.OP_LOGLIK_GRAD, P.OP_PREDICT):
        b = [P.workspace_bytes(m, n, dtype, op) for n in ns]
        assert all(x <= y for x, y in zip(b, b[1:])), op
    o16 = P.make_options(chunk=16)
    for n in ns:
        if P.workspace_bytes(m, n, dtype, P.OP_LOGLIK, o16) <= P.STATIC_SCRATCH_BYTES:
            assert P.workspace_bytes(m, n, dtype, P.OP_LOGLIK) <= P.STATIC_SCRATCH_BYTES, n


@pytest.mark.parametrize("chunk", [0, 100])
@pytest.mark.parametrize("dtype", [P.F32, P.F64])
@pytest.mark.parametrize("J", [1, 2, 3])
def test_quasiperiodic_workspace_monotone(J, dtype, chunk):
    """Chunks and the smoother's sub-chunks both follow from n."""
    m = P.make_model([(5, J, 1.0, 1.0, 1.0, 50.0), (MATERN32, 0, 20.0, 0.3)], 0.01)
    o = P.make_options(chunk=chunk) if chunk else None
    rng = np.random.default_rng(6)
    ns = set(int(v) for v in np.exp(rng.uniform(0, np.log(2e6), 400)))
    for q in (4096 * 16, 2048 * 64, 256 * 4096 // 3, 256 * 2048, 100 * 4096 // 5):
        ns |= {q + j for j in (-1, 0, 1)}
    ns = sorted(n for n in ns if n > 0)
    for op in (P.OP_LOGLIK, P.OP_PREDICT):
        b = [P.workspace_bytes(m, n, dtype, op, o) for n in ns]
        assert all(x <= y for x, y in zip(b, b[1:])), op


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 255, 257, 262144, 262145, 1048577])
def test_default_equals_explicit(n):
    if not gpu_available():
        pytest.skip("needs a HIP device")
    import torch
    m = P.make_model(MODELS["m32"], 0.01)
    g = torch.Generator(device="cuda").manual_seed(n)
    t = torch.cumsum(torch.rand(n, generator=g, device="cuda", dtype=torch.float64).cpu(), 0).cuda() * 0.02
    y = torch.sin(t) + 0.1 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    a = P.predict(m, t, y, dtype="float64")
    b = P.predict(m, t, y, dtype="float64", options=P.make_options(chunk=_expected(n, 65536)))
    for k in ("f_mean", "f_var", "loglik"):
        assert torch.equal(a[k], b[k]), k
    assert P.status(a["ws"]) == 0
