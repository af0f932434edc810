"""GPU parity of the training-side losses (spec_entropy_loss, spec_smooth_l1) against oracle/losses.py, through the
C-ABI.  Inputs are bf16-rounded before either side sees them; the library accumulates scores in fp32 and rounds
dL/ds to bf16 for its second product, so entropies are held to 1e-3 (the bar of the inference indicator) and
gradients to the bf16 bar of the forward tests (max-rel 2e-2 over the tensor)."""
import numpy as np
import pytest

from synth import gen
from synth.configs import DT_BF16, DT_F32
from tests.harness import build_case, make_ctx, rel_inf

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    case = build_case("ln-gelu-bf16", seed=3)
    c = make_ctx(case)
    yield c
    c.close()


def _inputs(seed, B, H, Hkv, R, dh, std):
    q = gen.normal(seed, f"q{B}{H}{R}{dh}", (B, H, R, dh), std, DT_BF16)
    k = gen.normal(seed, f"k{B}{Hkv}{R}{dh}", (B, Hkv, R, dh), std, DT_BF16)
    return q, k


@pytest.mark.parametrize("B,H,Hkv,R,dh,std", [
    (1, 1, 1, 1, 32, 1.0),          # a single row: H = 0, no gradient
    (2, 2, 2, 32, 64, 1.0),         # exactly one tile
    (2, 3, 3, 33, 64, 1.5),         # ragged tail of one row
    (1, 4, 2, 95, 32, 1.0),         # grouped heads, ragged
    (2, 5, 1, 70, 128, 0.7),        # 5:1 groups, head dim 128
    (3, 4, 4, 256, 64, 1.2),        # several tiles, the sequence length of the 256-token setting
    (1, 2, 2, 300, 64, 2.0),        # peaky rows
    (32, 16, 16, 256, 64, 1.0),     # the shape kernel_bench times (draft of configs[1]: 16 heads, 256 tokens)
])
def test_entropy_loss_and_gradients_match_oracle(ctx, B, H, Hkv, R, dh, std):
    from oracle import losses
    q, k = _inputs(5, B, H, Hkv, R, dh, std)
    loss, hr, dq, dk = ctx.spec_entropy_loss(ctx.dev_store(q), ctx.dev_store(k))
    ctx.sync()
    lo, hro, dqo, dko = losses.attn_entropy_loss(q, k)
    eh = float(np.abs(hr.cpu().numpy() - hro).max())
    el = abs(float(loss.item()) - lo)
    print(f"H rows {eh:.2e} (range {hro.min():.2f}..{hro.max():.2f}), loss {el:.2e}")
    assert eh < 1e-3
    assert el < 1e-4
    if R > 1:
        eq, ek = rel_inf(dq.cpu().numpy(), dqo), rel_inf(dk.cpu().numpy(), dko)
        print(f"dq {eq:.2e} dk {ek:.2e}")
        assert eq < 2e-2 and ek < 2e-2
    else:
        # a single column: Omega = 1 up to the rounding of s - ln sum exp in fp32
        assert np.abs(dq.cpu().numpy()).max() < 1e-6 and np.abs(dk.cpu().numpy()).max() < 1e-6


@pytest.mark.parametrize("B,H,Hkv,R,dh", [
    (1, 2, 1, 63, 128), (2, 2, 2, 65, 32),       # one row short of, and past, a 64-row tile of the walk
    (1, 3, 1, 127, 64), (2, 4, 2, 128, 128), (1, 2, 2, 129, 32),   # around the 128 rows of a workgroup
    (1, 4, 1, 385, 128),                         # an odd number of row groups, grouped heads
    (1, 1, 1, 1, 32), (3, 3, 1, 7, 64), (2, 5, 5, 31, 128), (5, 2, 1, 32, 32), (1, 6, 2, 24, 128),   # up to 32 rows: four heads a workgroup
    (1, 6, 2, 33, 128),                          # just above
])
def test_entropy_loss_around_tile_edges(ctx, B, H, Hkv, R, dh):
    """Same bars as above."""
    from oracle import losses
    q, k = _inputs(15, B, H, Hkv, R, dh, 1.0)
    loss, hr, dq, dk = ctx.spec_entropy_loss(ctx.dev_store(q), ctx.dev_store(k))
    ctx.sync()
    lo, hro, dqo, dko = losses.attn_entropy_loss(q, k)
    assert float(np.abs(hr.cpu().numpy() - hro).max()) < 1e-3
    assert abs(float(loss.item()) - lo) < 1e-4
    assert rel_inf(dq.cpu().numpy(), dqo) < 2e-2 and rel_inf(dk.cpu().numpy(), dko) < 2e-2


@pytest.fixture(scope="module")
def ctx_f32():
    c = make_ctx(build_case("ln-gelu-f32", seed=3))
    yield c
    c.close()


# below and above the size from which 16 bytes a lane are taken (1048576 bf16, 524288 float32 elements), tails after the last piece,
# inputs that start inside a piece (one element at a time there), and more than one step of the grid on every path
_L1_BF16 = [(7, 0), (8, 0), (4099, 0), (4099, 1), (4096, 3), (600001, 1), (1048583, 0), (1048584, 0), (4300003, 0)]
_L1_F32 = [(5, 0), (4099, 0), (600001, 1), (524291, 0), (524292, 0), (2200003, 0)]


@pytest.mark.parametrize("kind,n,shift", [("bf16", *c) for c in _L1_BF16] + [("f32", *c) for c in _L1_F32])
def test_smooth_l1_tails_and_unaligned_inputs(request, kind, n, shift):
    """Sums of positive float32 terms, at most 16 in a lane and then 20 levels of partial sums: below 36 x 2^-24; bar 1e-5."""
    from oracle import losses
    ctx, dt = (request.getfixturevalue("ctx"), DT_BF16) if kind == "bf16" else (request.getfixturevalue("ctx_f32"), DT_F32)
    p, t = gen.normal(16, f"p{n}", (n + shift,), 1.0, dt), gen.normal(16, f"t{n}", (n + shift,), 1.0, dt)
    loss, dp = ctx.spec_smooth_l1(ctx.dev_store(p)[shift:], ctx.dev_store(t)[shift:])
    ctx.sync()
    lo, dpo = losses.smooth_l1(p[shift:], t[shift:])
    assert abs(float(loss.item()) - lo) < 1e-5 * max(1.0, abs(lo))
    assert rel_inf(dp.cpu().numpy(), dpo) < 1e-5


def test_smooth_l1_gradient_buffer_on_sixteen_bytes(ctx):
    """The wide path asks 16-byte alignment of the gradient: a buffer that starts in the middle of 32 bytes, its neighbours intact."""
    from oracle import losses
    from paper_2512_08537_amd import binding
    import torch
    n = 1048584
    p, t = gen.normal(18, "p", (n,), 1.0, DT_BF16), gen.normal(18, "t", (n,), 1.0, DT_BF16)
    dp_, dt_ = ctx.dev_store(p), ctx.dev_store(t)
    buf, loss = torch.full((n + 8,), 7.0, device="cuda:0"), torch.zeros(1, device="cuda:0")
    assert buf[4:].data_ptr() % 32 == 16
    torch.cuda.synchronize()
    assert binding.lib.spec_smooth_l1(ctx.h, dp_.data_ptr(), dt_.data_ptr(), n, 1.0, loss.data_ptr(), buf[4:].data_ptr()) == 0
    ctx.sync()
    got = buf.cpu().numpy()
    assert rel_inf(got[4:n + 4], losses.smooth_l1(p, t)[1]) < 1e-5
    assert (got[:4] == 7.0).all() and (got[n + 4:] == 7.0).all()


def test_entropy_loss_outputs_are_optional_and_errors(ctx):
    from paper_2512_08537_amd.binding import FardError
    from oracle import losses
    q, k = _inputs(6, 1, 2, 2, 40, 64, 1.0)
    qd, kd = ctx.dev_store(q), ctx.dev_store(k)
    loss, hr, dq, dk = ctx.spec_entropy_loss(qd, kd, want_rows=False, want_dq=False, want_dk=True)
    ctx.sync()
    lo, _, _, dko = losses.attn_entropy_loss(q, k)
    assert hr is None and dq is None
    assert abs(float(loss.item()) - lo) < 1e-4
    assert rel_inf(dk.cpu().numpy(), dko) < 2e-2
    with pytest.raises(FardError):
        ctx.spec_entropy_loss(ctx.dev_store(q[..., :48]), ctx.dev_store(k[..., :48]))      # head dim 48
    with pytest.raises(FardError):
        ctx.spec_entropy_loss(ctx.dev_store(np.concatenate([q, q[:, :1]], axis=1)), kd)     # 3 heads over 2 kv heads


def test_entropy_loss_needs_a_bf16_context():
    from paper_2512_08537_amd.binding import FardError
    case = build_case("ln-gelu-f32", seed=3)
    c = make_ctx(case)
    x = c.dev_f32(np.zeros((1, 1, 32, 64), np.float32))
    with pytest.raises(FardError) as e:
        c.spec_entropy_loss(x, x)
    assert "FARD_ESTATE" in str(e.value)
    c.close()


@pytest.mark.parametrize("n,beta", [(1, 1.0), (257, 0.5), (100003, 1.0), (300000, 0.05)])
def test_smooth_l1_matches_oracle(ctx, n, beta):
    from oracle import losses
    p = gen.normal(7, f"p{n}", (n,), 1.0, DT_BF16)
    t = gen.normal(7, f"t{n}", (n,), 1.0, DT_BF16)
    loss, g = ctx.spec_smooth_l1(ctx.dev_store(p), ctx.dev_store(t), beta=beta)
    ctx.sync()
    lo, go = losses.smooth_l1(p, t, beta)
    assert float(loss.item()) == pytest.approx(lo, rel=2e-5)
    # elements within rounding of the kink may sit on either branch: both branches agree there to O(eps)
    assert np.allclose(g.cpu().numpy(), go, rtol=1e-5, atol=1e-6 / n)
