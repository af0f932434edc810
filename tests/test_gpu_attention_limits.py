"""NaN and infinite scores in the cached attention: a NaN key shows in every row that sees it, a key whose score is -inf has no
weight, and neither touches another sample.  Over the forms of the bf16 kernel (appending, without append, keys split over
workgroups, passes of rows) and the fp32 one, with the key in a block that every row sees whole and in the masked one."""
import numpy as np
import pytest

from tests.harness import build_case, make_ctx, rel_inf
from synth import configs

pytestmark = pytest.mark.gpu


def _rope_short():
    rc = configs.reduced("gqa-rope-bf16")                  # (a short cache: keys are not split over workgroups)
    rc.max_ctx, rc.n_ctx = 96, 70
    return rc


# name -> (configuration, rows of sample 0)
FORMS = {
    "append": (lambda: configs.reduced("ln-gelu-bf16"), 5),
    "append-64-wide": (lambda: configs.reduced("mid-bf16"), 9),
    "passes": (lambda: configs.reduced("mid-bf16"), 80),
    "rope": (_rope_short, 9),
    "rope-split": (lambda: configs.reduced("gqa-rope-bf16"), 9),
    "rope-passes": (lambda: configs.reduced("gqa-rope-bf16"), 30),
    "f32": (lambda: configs.reduced("ln-gelu-f32"), 5),
}


def _forward(case, n0):
    ctx = make_ctx(case)
    rows = np.concatenate([[n0], np.full(case.B - 1, 3)]).astype(np.int32)
    x = np.random.default_rng(4).normal(size=(int(rows.sum()), case.rc.target.d_latent)).astype(np.float32)
    z, _, ha = ctx.spec_forward(0, ctx.dev_f32(x), rows, commit=False, want_h_attn=True)
    ctx.sync()
    out = z.float().cpu().numpy(), ha.cpu().numpy()
    ctx.close()
    return out


@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("tail", [False, True])
def test_nan_key_shows_in_every_row_that_sees_it(form, tail):
    make, n0 = FORMS[form]
    case = build_case(make(), seed=31)
    z0, _ = _forward(case, n0)
    assert np.isfinite(z0).all()
    k, v = case.cache_t[0]
    k = k.copy()
    k[0, 0, (case.n_ctx - 1 if tail else 5), 3] = np.nan   # (the last cached position shares its block with the new rows)
    case.cache_t[0] = (k, v)
    z, ha = _forward(case, n0)
    assert np.isnan(z[:n0]).all()
    assert rel_inf(z[n0:], z0[n0:]) < 1e-2                 # (many rows: residual products of several K slices meet by atomics)
    assert np.isfinite(ha[n0:]).all()


@pytest.mark.parametrize("form", ["append", "append-64-wide", "passes"])
@pytest.mark.parametrize("keys", [slice(5, 6), slice(0, 32), slice(33, 36)])
def test_key_of_score_minus_infinity_has_no_weight(form, keys):
    """Queries of ones (zero weights, unit bias) against keys of -3e38, whose products sum to -inf in fp32: rows and row
    entropies of the first layer are those of a finite score far below every other one.  (Scores of 1e31 are also where a
    reference and a score that are rounded apart would be powers of two apart.)"""
    make, n0 = FORMS[form]
    out = []
    for low in (-3e38, -1e30):
        case = build_case(make(), seed=32)
        t = case.rc.target
        q = t.n_heads * t.d_head
        case.W["target.L0.wqkv"][:, :q] = 0.0
        case.W["target.L0.bqkv"][:q] = 1.0
        k, v = case.cache_t[0]
        k = k.copy()
        k[0, :, keys, :] = low
        case.cache_t[0] = (k, v)
        out.append(_forward(case, n0))
    (z, ha), (zf, haf) = out
    assert np.isfinite(zf).all() and np.isfinite(haf).all()
    assert rel_inf(z, zf) < 1e-2
    assert np.abs(ha - haf).max() < 1e-4
