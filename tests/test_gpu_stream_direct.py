"""GPU: streamed mode on pinned memory without copies (the default) against the
copies through staging slots (SDP_STREAM_DIRECT=0) and device mode, bit for
bit, over segments with ragged ends, rank counts on both sides of the stored
mean gradient's shapes, both gradient policies and several chunk sizes."""
import numpy as np
import pytest

import oracle
from gpu_util import DevState, HostState, check_state, hp_pair, log, need_gpu, rand_inputs, states_equal, torch

pytestmark = pytest.mark.gpu

TILE = 65536


@pytest.fixture(scope="module")
def sdp():
    return need_gpu()


@pytest.mark.parametrize("R", [1, 2, 3, 4, 6, 8, 16])
@pytest.mark.parametrize("never", [False, True])
def test_direct_equals_copies_and_device(sdp, R, never, monkeypatch):
    log(f"stream direct R={R} never={never}")
    sizes = [5 * TILE + 13, 1, 3, TILE, 4097]
    masters, grads = rand_inputs(sizes, R, 2, seed=77 + R)
    ref = oracle.State(masters)
    flags = sdp.SDP_FLAG_STREAM_GBAR_NEVER if never else 0

    def steps(direct, chunk):
        monkeypatch.setenv("SDP_STREAM_DIRECT", "1" if direct else "0")
        c = sdp.sdp_ctx_create(0, 4 * TILE, R, flags)
        st = HostState(sdp, masters, R)
        norms = []
        try:
            for t in (1, 2):
                st.set_grads(grads[t - 1])
                hs, _ = hp_pair(sdp, lr=1e-3, weight_decay=0.02, max_grad_norm=0.05, step=t)
                norms.append(sdp.sdp_stream_step(c, st.segments(), hs, chunk))
                assert sdp.sdp_grad_norm(c, st.segments(), False, chunk) == norms[-1]
            return st.host(), norms
        finally:
            st.close()
            sdp.sdp_ctx_destroy(c)

    dev = DevState(masters, R)
    c = sdp.sdp_ctx_create(0, 0, R, 0)
    want = []
    try:
        for t in (1, 2):
            hs, ho = hp_pair(sdp, lr=1e-3, weight_decay=0.02, max_grad_norm=0.05, step=t)
            dev.set_grads(grads[t - 1])
            want.append(sdp.sdp_agg_adam_step(c, dev.segments(sdp), hs, 0, torch.cuda.current_stream(), want_norm=True))
            assert want[-1] == oracle.step(ref, grads[t - 1], ho)[1]
    finally:
        sdp.sdp_ctx_destroy(c)
    base = dev.host()
    check_state(base, ref)
    for direct, chunk in ((True, TILE), (True, 4 * TILE), (False, TILE), (False, 3 * TILE), (False, 4 * TILE)):
        got, norms = steps(direct, chunk)
        assert norms == want, (direct, chunk)
        assert states_equal(got, base), (direct, chunk)


def test_pinned_memory_takes_the_direct_path(sdp, monkeypatch):
    """sdp_host_alloc's memory is known to the runtime as one allocation, so
    the direct path takes it: one launch of each kernel, where copies make one
    per chunk."""
    n, R = 3 * TILE + 5, 2
    masters, grads = rand_inputs([n], R, 1, seed=9)
    st = HostState(sdp, masters, R)
    st.set_grads(grads[0])
    launches = []
    try:
        for direct in ("1", "0"):
            monkeypatch.setenv("SDP_STREAM_DIRECT", direct)
            c = sdp.sdp_ctx_create(0, TILE, R, 0)
            try:
                sdp.sdp_ctx_set_timing(c, True)
                sdp.sdp_stream_step(c, st.segments(), sdp.make_params(step=1), TILE)
                t = sdp.sdp_ctx_get_timing(c)
                launches.append((t.norm_launches, t.update_launches))
            finally:
                sdp.sdp_ctx_destroy(c)
    finally:
        st.close()
    assert launches[0] == (1, 1) and launches[1][1] == 4, launches


def test_direct_non_finite_leaves_states(sdp):
    n, R = TILE + 9, 3
    masters, grads = rand_inputs([n], R, 1, seed=5)
    grads[0][0][1][7] = 0x7f80  # +inf
    st = HostState(sdp, masters, R)
    st.set_grads(grads[0])
    before = st.host()
    c = sdp.sdp_ctx_create(0, TILE, R, 0)
    try:
        with pytest.raises(sdp.SdpNonFinite):
            sdp.sdp_stream_step(c, st.segments(), sdp.make_params(step=1), TILE)
        assert states_equal(before, st.host())
    finally:
        st.close()
        sdp.sdp_ctx_destroy(c)
