"""GPU: the streamed calls on pinned memory wait for the host link, and leave
the compute units to other work meanwhile.  A matrix product on another stream
(a kernel that needs LDS) runs beside them; its latency must stay far below the
time that the norm pass alone takes, which it would wait out if the pass held
the LDS of every compute unit."""
import threading
import time

import numpy as np
import pytest

from gpu_util import log, need_gpu, torch

pytestmark = pytest.mark.gpu

TILE = 65536


@pytest.fixture(scope="module")
def sdp():
    return need_gpu()


@pytest.mark.parametrize("R", [4, 8])
@pytest.mark.parametrize("call", ["step", "norm"])
def test_other_streams_run_beside_a_streamed_call(sdp, R, call):
    log(f"beside streamed {call} R={R}")
    n = 64 << 20  # the norm pass reads 0.5 or 1 GB: 9 or 18 ms at 57 GB/s
    bufs = [sdp.HostBuffer(n * size) for size in (4, 4, 4, 2) + (2,) * R]
    for b in bufs[:3]:
        b.view(np.float32, n)[:] = 0.01
    for b in bufs[3:]:
        b.view(np.uint16, n)[:] = 0x3a00
    segs = sdp.Segments([(bufs[0].ptr, bufs[1].ptr, bufs[2].ptr, bufs[3].ptr, [b.ptr for b in bufs[4:]], n)])
    hp = sdp.make_params(step=100)
    a = torch.randn(4096, 4096, device="cuda", dtype=torch.bfloat16)
    # the process has four hardware queues; a stream that shares the context's
    # waits for its kernels whatever they hold, so the best of four is judged
    streams = [torch.cuda.Stream() for _ in range(4)]

    def product(side):
        t = time.perf_counter()
        with torch.cuda.stream(side):
            torch.mm(a, a)
        side.synchronize()
        return (time.perf_counter() - t) * 1e3
    torch.cuda.synchronize()
    for side in streams:
        for _ in range(3):
            product(side)
    ctx = sdp.sdp_ctx_create(0, TILE, R, 0)

    def streamed():
        if call == "step":
            sdp.sdp_stream_step(ctx, segs, hp, TILE)
        else:
            sdp.sdp_grad_norm(ctx, segs, False, TILE)
    try:
        streamed()
        norm_ms = 2 * R * n / 57e6
        best = None
        for side in streams:
            worker = threading.Thread(target=lambda: [streamed() for _ in range(4)])
            beside = []
            worker.start()
            while worker.is_alive():
                beside.append(product(side))
            worker.join()
            # a product takes 0.14 ms alone; one may be held up by the host's scheduling
            slow = sum(x > norm_ms / 2 for x in beside)
            log(f"beside streamed {call} R={R}: {len(beside)} products, median {np.median(beside):.3f} ms, "
                f"largest {max(beside):.3f} ms, {slow} slow; norm pass {norm_ms:.1f} ms")
            if best is None or len(beside) > best[0]:
                best = len(beside), slow
        assert best[0] >= 40 and best[1] <= 1
    finally:
        sdp.sdp_ctx_destroy(ctx)
