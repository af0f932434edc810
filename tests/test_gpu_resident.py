"""Head decodes whose workgroups wait for one another (resident launches): when they are used, what turns them off, and what a
launch that waits in vain leaves behind."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import head as ohd
from paper_2512_08537_amd import binding
from synth import gen
from synth.configs import HeadCfg, RoundCfg, TfCfg
from tests.harness import build_case, gpu_inputs, make_ctx, rel_inf, to_np

pytestmark = pytest.mark.gpu


def _case(w, seed=9, blocks=3, steps=2):
    tf = TfCfg(n_layers=1, d_model=128, n_heads=2, n_kv_heads=2, d_head=64, d_ff=256, max_pos=32)
    rc = RoundCfg(name="resident", target=tf, draft=tf, head=HeadCfg(blocks, w, 128, n_steps=steps), K=8, max_batch=16, max_ctx=32,
                  entropy_layer=1, batch=4, n_ctx=8)
    return build_case(rc, seed=seed)


def _inputs(case, n, seed=17):
    h = case.rc.head
    return gen.normal(seed, f"z{n}", (n, h.d_cond), 1.0, case.rc.dtype), gen.noise(seed, f"e{n}", (h.n_steps + 1, n, h.d_latent))


def _decode(ctx, z, eps):
    mu, x = ctx.diffhead_decode(ctx.dev_store(z), ctx.dev_f32(eps))
    ctx.sync()
    return mu.cpu().numpy(), x.cpu().numpy()


def _check(case, got, z, eps):
    mu_o, x_o = ohd.decode(case.rc.head, case.W, z, eps)
    assert rel_inf(got[0], mu_o) < 2e-2 and rel_inf(got[1], x_o) < 2e-2


@pytest.mark.parametrize("w,tiles", [(1024, {1: 1, 32: 1, 33: 2, 64: 2, 65: 0}), (1280, {1: 1, 16: 1, 17: 2, 48: 2, 49: 0}),
                                     (1536, {1: 1, 16: 1, 17: 0}), (512, {1: 0, 16: 0})])
def test_which_decodes_are_resident(w, tiles):
    """Row limits with four launches side by side, fewer rows with eight, none with 0, and the limits of init again."""
    ctx = make_ctx(_case(w))
    assert {n: ctx.spec_resident_tiles(n) for n in tiles} == tiles
    ctx.spec_resident(launches=8)
    for n in (1, 16, 17, 32, 33, 48, 49, 64):
        t = ctx.spec_resident_tiles(n)
        assert t == 0 or w // (16 * t) * -(-n // 16) * 8 <= 2 * 256
    assert ctx.spec_resident_tiles(max(tiles)) == 0
    ctx.spec_resident(launches=0)
    assert ctx.spec_resident_tiles(1) == 0
    ctx.spec_resident(launches=4)
    assert {n: ctx.spec_resident_tiles(n) for n in tiles} == tiles
    ctx.spec_resident(launches=1)                          # (room for more rows than init reserved words for: not taken)
    assert ctx.spec_resident_tiles(max(tiles)) == 0
    with pytest.raises(binding.FardError) as e:
        ctx.spec_resident(give_up_s=21.0)
    assert e.value.code == -1
    ctx.close()


def test_switched_off_it_is_a_launch_per_product():
    case = _case(1024)
    ctx = make_ctx(case)
    z, eps = _inputs(case, 33)
    on = _decode(ctx, z, eps)
    ctx.spec_resident(launches=0)
    off = _decode(ctx, z, eps)
    _check(case, on, z, eps)
    _check(case, off, z, eps)
    assert not np.array_equal(on[0], off[0])               # (other tiles, other sums: another path did run)
    ctx.close()


@pytest.mark.parametrize("w,n", [(1024, 4), (1024, 8), (1024, 16), (1024, 64), (1280, 48), (1536, 16)])
def test_launch_that_waits_in_vain_is_reported(w, n):
    """Launches short of one workgroup, whose words never come: every other one gives up after a millisecond and exits, the rows
    are NaN, later launches do not wait, the next call says so once, and the context goes on without."""
    case = _case(w)
    ctx = make_ctx(case)
    z, eps = _inputs(case, n)
    good = _decode(ctx, z, eps)
    _check(case, good, z, eps)
    ctx.spec_resident(give_up_s=0.0)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    mu, x = ctx.diffhead_decode(ctx.dev_store(z), ctx.dev_f32(eps))
    b.record()
    ctx.sync()
    assert torch.isnan(mu).all() and torch.isnan(x).all()
    assert a.elapsed_time(b) < 500.0
    with pytest.raises(binding.FardError) as e:
        ctx.spec_kv_lengths(binding.TARGET, 4)
    assert e.value.code == -5 and "waited too long" in str(e.value)
    assert ctx.spec_resident_tiles(n) == 0
    _check(case, _decode(ctx, z, eps), z, eps)
    ctx.spec_resident(launches=4, give_up_s=10.0)          # the user has mended the cause: the path can be had again
    assert ctx.spec_resident_tiles(n) > 0
    again = _decode(ctx, z, eps)
    assert np.array_equal(again[0], good[0]) and np.array_equal(again[1], good[1])
    ctx.close()


@pytest.mark.parametrize("graph", [False, True])
def test_rounds_after_a_launch_that_waited_in_vain(graph):
    """A round whose head launches give up fails, or the call behind it; the next round on restored caches is that of a context
    without resident launches, and with them allowed again that of before, also recorded and replayed."""
    case = _case(1024)
    ctx = make_ctx(case, stream=torch.cuda.Stream())
    inp = gpu_inputs(ctx, case)
    torch.cuda.synchronize()

    def one():
        for which in (binding.TARGET, binding.DRAFT):
            ctx.spec_kv_reset(which, np.full(case.B, case.n_ctx, dtype=np.int32))
        out = ctx.spec_round(inp["pending"], inp["eps"], inp["r"], 0.0, out=bufs)
        ctx.sync()
        return to_np(out)

    bufs = ctx._round_bufs(case.B)
    if graph:
        ctx.spec_graph_enable(True)
    with_path = [one() for _ in range(4)]
    ctx.spec_resident(launches=0)
    without = [one() for _ in range(4)]
    ctx.spec_resident(launches=4, give_up_s=0.0)
    with pytest.raises(binding.FardError) as e:
        one()
        ctx.spec_kv_lengths(binding.TARGET, case.B)
    assert e.value.code == -5
    ctx.sync()
    after = [one() for _ in range(4)]
    ctx.spec_resident(launches=4, give_up_s=10.0)
    again = [one() for _ in range(4)]
    for key in ("mu_p", "x_draft", "n_accept", "log_ratio"):
        assert np.isfinite(with_path[0][key]).all()
        assert all(np.array_equal(a[key], with_path[0][key]) for a in with_path + again)
        assert all(np.array_equal(a[key], without[0][key]) for a in without + after)
    ctx.close()


@pytest.mark.parametrize("w,n", [(1024, 64), (1280, 48), (1536, 16)])
def test_contexts_on_streams_of_their_own_decode_at_once(w, n):
    """Three contexts at the row limit, decodes of all in flight together: the results of each alone."""
    cases = [_case(w, seed=20 + i) for i in range(3)]
    streams = [torch.cuda.Stream() for _ in cases]
    ctxs = [make_ctx(c, stream=s) for c, s in zip(cases, streams)]
    io = []
    for c, ctx in zip(cases, ctxs):
        z, eps = _inputs(c, n, seed=c.seed)
        io.append((ctx.dev_store(z), ctx.dev_f32(eps)))
        assert ctx.spec_resident_tiles(n) > 0
    def run(i, out):
        z, eps = io[i]
        assert binding.lib.diffhead_decode(ctxs[i].h, z.data_ptr(), None, n, eps.data_ptr(), out[0].data_ptr(), out[1].data_ptr()) == 0

    # (outputs are filled on torch's stream: all of them before the first decode)
    alone = [torch.full((2, n, 16), -7.0, device="cuda") for _ in ctxs]
    outs = [torch.full((20, 2, n, 16), -7.0, device="cuda") for _ in ctxs]
    torch.cuda.synchronize()
    for i, out in enumerate(alone):
        run(i, out)
        torch.cuda.synchronize()
    for k in range(20):
        for i in range(len(ctxs)):
            run(i, outs[i][k])
    torch.cuda.synchronize()
    for i, (case, ctx) in enumerate(zip(cases, ctxs)):
        assert all(torch.equal(out, alone[i]) for out in outs[i])
        ctx.spec_kv_lengths(binding.TARGET, 4)             # (nothing gave up)
        z, eps = _inputs(case, n, seed=case.seed)
        _check(case, [t.cpu().numpy() for t in alone[i]], z, eps)
        ctx.close()


@pytest.mark.parametrize("w", [1024, 1280, 1536])
@pytest.mark.parametrize("n,between", [(8, 1), (16, 3), (4, 16), (16, 8)])
def test_tags_that_start_over_match_no_word_of_before(w, n, between):
    """A head of one block and one step uses every exchange buffer once a decode, so its words stay with their first tags.  A decode
    of n rows, one of another row count in which the count of decodes passes a multiple of 2^20, and a decode of other values
    whose tags are those of the first."""
    case = _case(w, blocks=1, steps=1)
    first, mid, last = _inputs(case, n, seed=1), _inputs(case, between, seed=2), _inputs(case, n, seed=3)
    for turn in (1, 4096):                                 # (the second: the count itself wraps)
        ctx = make_ctx(case)
        ctx.spec_resident(decodes=(turn - 1) << 20)
        _check(case, _decode(ctx, *first), *first)
        ctx.spec_resident(decodes=(turn << 20) - 1)
        _check(case, _decode(ctx, *mid), *mid)
        _check(case, _decode(ctx, *last), *last)
        ctx.close()


class _Stream:
    def __init__(self, ptr):
        self.cuda_stream = ptr


def test_stream_with_a_mask_takes_a_launch_per_product():
    """All compute units but one: the count of workgroups that fit the chip does not hold for the stream."""
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = C.CDLL(path)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    words = (C.c_uint32 * ((units + 31) // 32))(*[0xFFFFFFFF] * ((units + 31) // 32))
    words[len(words) - 1] = (1 << ((units - 1) % 32)) - 1
    stream = C.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(C.byref(stream), len(words), words) == 0
    case = _case(1024)
    ctx = make_ctx(case, stream=_Stream(stream.value))
    assert ctx.spec_resident_tiles(1) == 0
    ctx.spec_resident(launches=1)
    assert ctx.spec_resident_tiles(1) == 0
    z, eps = _inputs(case, 49)
    _check(case, _decode(ctx, z, eps), z, eps)
    ctx.close()
    torch.cuda.synchronize()
    assert hip.hipStreamDestroy(stream) == 0
