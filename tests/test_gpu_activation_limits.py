"""GELU and SiLU of the bf16 epilogues where their divisions meet the end of the fp32 range, at infinities and NaN."""
import numpy as np
import pytest
import torch

from oracle import transformer as otf
from synth import gen
from tests.harness import build_case, make_ctx

pytestmark = pytest.mark.gpu

VALUES = np.concatenate([np.arange(-96.0, -79.0, 0.5), np.linspace(-79.0, 79.0, 317), np.arange(80.0, 96.0, 0.5),
                         [0.0, -0.0, 1e-30, -1e-30, 1e-38, -1e-38, 1e30, -1e30, 3e38, -3e38, np.inf, -np.inf, np.nan]])


@pytest.fixture(scope="module")
def ctx():
    c = make_ctx(build_case("ln-gelu-bf16", seed=0))
    yield c
    c.close()


@pytest.mark.parametrize("route,K", [("narrow", 1024), ("narrow", 192), ("gemm", 1024), ("gemm", 192)])
@pytest.mark.parametrize("act", [1, 2])
def test_activation_over_the_whole_range(ctx, route, K, act):
    """Rows of one value and zeros against a first weight row of ones: the accumulator is the value itself.  SiLU: half an ulp of
    bf16 and the exponential's error, down to x = -88.7 where e^-x leaves fp32 (0 beyond: as x / inf); GELU: the published error
    of its erf, 1.5e-7, times |x| / 2 on top.  At infinities what the formulas give: -inf has no limit there, and neither has NaN."""
    x = gen.bf16_round(VALUES.astype(np.float32))
    if route == "gemm":
        x = np.tile(x, 4)                                  # (many rows: the streaming or LDS-tiled kernels)
    N = 1024
    A = np.zeros((len(x), K), np.float32)
    A[:, 0] = x
    W = np.zeros((K, N), np.float32)
    W[0] = 1.0
    dA, dW = ctx.dev_store(A), ctx.dev_store(W)
    if route == "narrow":
        out = ctx.spec_gemm_narrow(dA, dW, ctx.empty((len(x), N), torch.bfloat16), epi=0, act=act)
    else:
        out = ctx.spec_gemm(dA, dW, act=act)
    ctx.sync()
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.array_equal(got, np.repeat(got[:, :1], N, axis=1), equal_nan=True)
    got, v = got[:, 0], x.astype(np.float64)
    assert np.isnan(got[np.isnan(v) | (v == -np.inf)]).all() and (got[v == np.inf] == np.inf).all()
    fin = np.isfinite(v)
    got, v = got[fin], v[fin]
    with np.errstate(over="ignore"):
        ref = np.where(v < -88.72, 0.0, otf.silu(v)) if act == 2 else otf.gelu_erf(v)
    bar = 2.0 ** -8 * np.abs(ref) + (2e-7 * np.minimum(np.abs(v), 16.0) if act == 1 else 0.0) + 1e-40
    assert (np.abs(got - ref) <= bar).all(), [(a, b, c) for a, b, c, d in zip(v, got, ref, bar) if abs(b - c) > d]
