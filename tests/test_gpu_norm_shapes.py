"""GPU: the norm pass at the edges of its spans and lane groups.  The sum of
squares is carried as a pair of FP64 numbers to at least 2^-85 of itself, so
its FP64 rounding, and with it the norm, is the oracle's, which rounds the
exact sum once; the comparison is therefore of bits."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import DevState, check_state, hp_pair, log, need_gpu, rand_inputs, torch

pytestmark = pytest.mark.gpu

# one-wave spans of 256, block spans of 4,096 and 8,192, groups of 4 and 8, tiles of 65,536
SIZES = [3, 255, 256, 257, 263, 4095, 4096, 4100, 8185, 8191, 8192, 8193, 65535, 65536 + 8193]


@pytest.fixture(scope="module")
def sdp():
    return need_gpu()


@pytest.mark.parametrize("R", [1, 2, 3, 4, 5, 6, 7, 8, 12, 16])
@pytest.mark.parametrize("store", [False, True])
def test_norm_bits_at_span_edges(sdp, R, store):
    log(f"norm shapes R={R} store={store}")
    ctx = sdp.sdp_ctx_create(0, 0, R, sdp.SDP_FLAG_DEVICE_GBAR_ALWAYS if store else sdp.SDP_FLAG_DEVICE_GBAR_NEVER)
    rng = np.random.default_rng(100 * R + store)
    try:
        for n in SIZES:
            masters, grads = rand_inputs([n], R, 1, seed=31 * n + R)
            for kind in ("normal", "wide", "zeros"):
                gs = [g.copy() for g in grads[0][0]]
                for g in gs:
                    if kind == "wide":  # binades from 2^-60 to 2^60, some lanes beyond the fast route's window
                        e = rng.integers(67, 188, n).astype(np.uint16) << 7
                        g[:] = e | (g & 0x807f)
                    elif kind == "zeros":
                        g[rng.random(n) < 0.5] = rng.choice([0, 0x8000])
                dev = DevState(masters, R)
                dev.set_grads([gs])
                hs, ho = hp_pair(sdp, lr=1e-3, weight_decay=0.02, max_grad_norm=0.05, step=3)
                ref = oracle.State(masters)
                _, onorm = oracle.step(ref, [gs], ho)
                s = torch.cuda.current_stream()
                norm = sdp.sdp_agg_adam_step(ctx, dev.segments(sdp), hs, 0, s, want_norm=True)
                assert norm == onorm, (n, kind, norm, onorm)
                assert sdp.sdp_grad_norm(ctx, dev.segments(sdp), True, 0, s) == onorm, (n, kind)
                check_state(dev.host(), ref)
    finally:
        sdp.sdp_ctx_destroy(ctx)


@pytest.mark.parametrize("R", [3, 4, 5, 6, 8, 12, 16])
@pytest.mark.parametrize("below", [20, 24, 28, 32])
def test_norm_bits_where_ranks_cancel(sdp, R, below):
    """Two ranks cancel and the others lie `below` binades under them, still
    inside the fast route's window: the sum of squares keeps its precision
    relative to the means, not to the gradients, so the pass that stores
    g_bar, the reading pass and the no-allocation entry point (whose spans and
    orders differ) all give the oracle's bits."""
    log(f"norm where ranks cancel R={R} below={below}")
    n = 65536 + 4099
    rng = np.random.default_rng(1000 * R + below)
    masters, _ = rand_inputs([n], R, 1, seed=R)
    hs, ho = hp_pair(sdp, lr=1e-3, weight_decay=0.02, max_grad_norm=0.05, step=3)
    s = torch.cuda.current_stream()
    stored = sdp.sdp_ctx_create(0, 0, R, sdp.SDP_FLAG_DEVICE_GBAR_ALWAYS)
    reading = sdp.sdp_ctx_create(0, 0, R, sdp.SDP_FLAG_DEVICE_GBAR_NEVER)
    try:
        for trial in range(6):
            big = synth.to_bf16_bits(rng.uniform(1, 2, n).astype(np.float32))
            gs = [big, big ^ 0x8000] + [synth.to_bf16_bits((rng.standard_normal(n) * 2.0 ** (-below - 5 * (k % 2))
                                                            ).astype(np.float32)) for k in range(R - 2)]
            ref = oracle.State(masters)
            _, onorm = oracle.step(ref, [gs], ho)
            for ctx in (stored, reading, None):
                dev = DevState(masters, R)
                dev.set_grads([gs])
                if ctx is None:
                    norm = sdp.sdp_agg_adam_step_noalloc(dev.segments(sdp), hs, s, want_norm=True)
                else:
                    norm = sdp.sdp_agg_adam_step(ctx, dev.segments(sdp), hs, 0, s, want_norm=True)
                    assert sdp.sdp_grad_norm(ctx, dev.segments(sdp), True, 0, s) == onorm, trial
                assert norm == onorm, (trial, ctx is None, norm, onorm)
                check_state(dev.host(), ref)
    finally:
        sdp.sdp_ctx_destroy(stored)
        sdp.sdp_ctx_destroy(reading)


@pytest.mark.parametrize("R", [1, 3, 4, 8, 16])
@pytest.mark.parametrize("count", [2, 19, 33, 64])
def test_many_segments(sdp, R, count):
    """Calls around the number of segments that one launch takes (19 to 32, by
    the rank count), with sizes around a lane's group, a block's groups and
    spans: device mode and the no-allocation entry point against the oracle."""
    log(f"many segments R={R} count={count}")
    sizes = [[1, 3, 4, 255, 256, 257, 1027, 4096, 5000, 8193, 20000][k % 11] for k in range(count)]
    sizes[count // 2] = 65536 + 5
    masters, grads = rand_inputs(sizes, R, 1, seed=7 * count + R)
    hs, ho = hp_pair(sdp, lr=1e-3, weight_decay=0.02, max_grad_norm=0.05, step=2)
    ref = oracle.State(masters)
    _, onorm = oracle.step(ref, grads[0], ho)
    s = torch.cuda.current_stream()
    ctx = sdp.sdp_ctx_create(0, 0, R, 0)
    try:
        for noalloc in (False, True):
            dev = DevState(masters, R)
            dev.set_grads(grads[0])
            if noalloc:
                norm = sdp.sdp_agg_adam_step_noalloc(dev.segments(sdp), hs, s, want_norm=True)
            else:
                norm = sdp.sdp_agg_adam_step(ctx, dev.segments(sdp), hs, 0, s, want_norm=True)
            assert norm == onorm, (noalloc, norm, onorm)
            check_state(dev.host(), ref)
    finally:
        sdp.sdp_ctx_destroy(ctx)


@pytest.mark.parametrize("R,n", [(2, 16 * 65536), (2, 16 * 65536 + 1), (3, 128 * 65536), (3, 128 * 65536 + 1),
                                 (8, 65536), (8, 65537), (8, 8 * 65536 + 1), (16, 70 * 65536), (1, 33 * 65536 - 3)])
def test_pair_counts_at_the_finalizes_edges(sdp, R, n):
    """256 pairs are summed by the update itself, up to 2,048 by one block of
    the finalize, more by several; three steps, so that the count of blocks is
    used again, and without reading the norm back in between."""
    log(f"finalize edges R={R} n={n}")
    masters, grads = rand_inputs([n], R, 1, seed=n % 1000 + R)
    ref = oracle.State(masters)
    s = torch.cuda.current_stream()
    ctx = sdp.sdp_ctx_create(0, 0, R, 0)
    try:
        dev, dev2 = DevState(masters, R), DevState(masters, R)
        dev.set_grads(grads[0])
        dev2.set_grads(grads[0])
        for t in (1, 2, 3):
            hs, ho = hp_pair(sdp, lr=1e-3, weight_decay=0.02, max_grad_norm=0.05, step=t)
            _, onorm = oracle.step(ref, grads[0], ho)
            norm = sdp.sdp_agg_adam_step(ctx, dev.segments(sdp), hs, 0, s, want_norm=t == 3)
            sdp.sdp_agg_adam_step_noalloc(dev2.segments(sdp), hs, s)
        assert norm == onorm
        assert sdp.sdp_ctx_last_norm(ctx)[0] == onorm
        check_state(dev.host(), ref)
        check_state(dev2.host(), ref)
    finally:
        sdp.sdp_ctx_destroy(ctx)


@pytest.mark.parametrize("R,sizes", [(16, [3125003]), (16, [3124997]), (16, [2000005, 1200003, 4099]), (1, [5, 70001])])
def test_calls_around_the_cache_rule(sdp, R, sizes):
    """The update re-reads gradients through the cache up to 50e6 / R elements
    and with the non-temporal hint above: both kernels, for one segment and for
    several, give the oracle's states."""
    log(f"cache rule R={R} sizes={sizes}")
    masters, grads = rand_inputs(sizes, R, 1, seed=sum(sizes) % 1000)
    hs, ho = hp_pair(sdp, lr=1e-3, weight_decay=0.02, max_grad_norm=0.05, step=2)
    ref = oracle.State(masters)
    _, onorm = oracle.step(ref, grads[0], ho)
    s = torch.cuda.current_stream()
    ctx = sdp.sdp_ctx_create(0, 0, R, sdp.SDP_FLAG_DEVICE_GBAR_NEVER)
    try:
        dev = DevState(masters, R)
        dev.set_grads(grads[0])
        assert sdp.sdp_agg_adam_step(ctx, dev.segments(sdp), hs, 0, s, want_norm=True) == onorm
        check_state(dev.host(), ref)
    finally:
        sdp.sdp_ctx_destroy(ctx)


def test_a_call_of_many_small_segments_does_not_wait(sdp):
    """Room for the span pairs of 4,096 tiles is there from the start, also
    where g_bar is stored with its 256 pairs per tile: an asynchronous call on
    many small segments returns while earlier work on the stream still runs."""
    log("many small segments, no wait")
    R, big, small, count = 8, 30_000_000, 20_000, 1000
    p, m, v = (torch.zeros(big, device="cuda") for _ in range(3))
    pb = torch.zeros(big, dtype=torch.int16, device="cuda")
    g = [torch.zeros(big, dtype=torch.int16, device="cuda") for _ in range(R)]
    cut = lambda a, n: (p[a:a + n], m[a:a + n], v[a:a + n], pb[a:a + n], [x[a:a + n] for x in g])
    hs = sdp.make_params(step=1)
    s = torch.cuda.current_stream()
    ctx = sdp.sdp_ctx_create(0, 0, R, 0)
    try:
        # the mean gradient's own room grows here
        sdp.sdp_agg_adam_step(ctx, sdp.segments_from_tensors([cut(0, big)]), hs, 0, s)
        segs = sdp.segments_from_tensors([cut(k * small, small) for k in range(count)])
        torch.cuda.synchronize()
        torch.cuda._sleep(400_000_000)  # a few tenths of a second
        slept = torch.cuda.Event()
        slept.record()
        sdp.sdp_agg_adam_step(ctx, segs, hs, 0, s)
        assert not slept.query(), "the call waited for the device"
        torch.cuda.synchronize()
    finally:
        sdp.sdp_ctx_destroy(ctx)
