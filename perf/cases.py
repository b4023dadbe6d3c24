"""The calls that this library's users make, for timing and comparison.

A training program calls the update once per iteration: on states in device
memory (device mode, or its no-allocation entry point inside captured or
allocation-free code), on states in pinned host memory streamed through the
GPU, or on the host-update route; and it delivers the updated parameters for
the next forward pass.  The listed cases are those calls over the sizes that
the library serves, from a few small tensors to a whole layer of the largest
model, with one flat segment per layer, a layer's tensors as segments of
their own, or a whole small model in one call.

A case is a dict of plain values:
  kind    "step" (sdp_agg_adam_step), "noalloc" (sdp_agg_adam_step_noalloc),
          "norm" (sdp_grad_norm on device gradients), "stream"
          (sdp_stream_step), "route" (sdp_host_update_step) or "deliver"
          (sdp_deliver_params)
  sizes   elements of each segment, comma-separated
  flat    the segments are pieces of shared flat buffers (true) or separate
          allocations (false)
  ranks   rank gradients per segment
  sigma, outliers   gradient distribution: N(0, sigma), a share of the
          elements 100 times larger
  want_norm  the caller reads the gradient norm back (and so waits)
  chunk   elements per chunk (stream, route, deliver)
  bf16    route: the mean gradient returns in BF16
"""
import weakref

import numpy as np
import torch

from paper_2609_34162_amd import sdp

DEV = "cuda:0"
TILE = 65536
STEP = 100          # the optimizer step t that every case takes
HP = dict(lr=1e-5, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01, max_grad_norm=1.0)
MASTER_SIGMA = 0.02
PIECE = 1 << 26     # elements generated or evaluated at a time
VOCAB = 151936


def layer_tensors(hidden, kv, ffn):
    """q/k/v/o, gate/up/down and the two norm vectors of a decoder layer."""
    return [hidden * hidden, kv * hidden, kv * hidden, hidden * hidden, ffn * hidden, ffn * hidden, hidden * ffn,
            hidden, hidden]


def case(kind, sizes, ranks, flat=True, sigma=1e-3, outliers=0.0, want_norm=False, chunk=0, bf16=False, name=None):
    c = dict(kind=kind, sizes=",".join(str(n) for n in sizes), ranks=ranks, flat=flat, sigma=sigma, outliers=outliers,
             want_norm=want_norm, chunk=chunk, bf16=bf16)
    if name:
        c["name"] = name
    return c


QWEN3_8B = sum(layer_tensors(4096, 1024, 12288))
QWEN25_72B = sum(layer_tensors(8192, 1024, 29568))


def listed():
    return [
        # a handful of small ragged tensors (adapters, norms, biases): the smallest call
        case("step", [2 * TILE + 3, 1, 100000, 8], 4, flat=False, outliers=0.01, want_norm=True,
             name="small_tensors_r4"),
        # one 1024 x 1024 weight, two ranks
        case("step", [1 << 20], 2, name="weight_1m_r2"),
        # a decoder layer whose nine tensors were never concatenated; the
        # program logs the norm of each step
        case("step", layer_tensors(2048, 512, 6144), 4, flat=False, outliers=0.01, want_norm=True,
             name="layer_tensors_48m_r4"),
        # a whole small model in one call, gradients already reduced by the
        # data-parallel library: embedding, 24 layers and head
        case("step", [VOCAB * 1024] + 24 * [sum(layer_tensors(1024, 512, 3072))] + [VOCAB * 1024], 1,
             name="model_616m_r1"),
        # one Qwen3-8B layer, gradients with outliers (the device workload)
        case("step", [QWEN3_8B], 4, outliers=0.01, name="qwen3_8b_layer_r4"),
        # one Qwen2.5-72B layer, eight ranks: the largest device call
        case("step", [QWEN25_72B], 8, sigma=5e-4, name="qwen2.5_72b_layer_r8"),
        # the entry point for callers that cannot allocate: a layer in two
        # odd-sized pieces, a rank count that is no power of two
        case("noalloc", [20000003, 4194301], 3, outliers=0.01, name="noalloc_24m_r3"),
        # gradient-norm monitoring alone
        case("norm", [100663303], 8, want_norm=True, name="grad_norm_101m_r8"),
        # states in pinned host memory: one Qwen3-8B layer in 16M-element chunks
        case("stream", [QWEN3_8B], 4, outliers=0.01, want_norm=True, chunk=16 << 20, name="stream_qwen3_8b_layer_r4"),
        # the same mode on a small layer, small chunks
        case("stream", [12595203, 4096], 2, want_norm=True, chunk=1 << 20, name="stream_13m_r2"),
        # the host-update route: gradients on the GPU, states in pageable host memory
        case("route", [QWEN3_8B], 4, outliers=0.01, want_norm=True, chunk=32 << 20, bf16=True,
             name="route_qwen3_8b_layer_r4"),
        # parameter delivery of an updated layer for the next forward pass
        case("deliver", [QWEN3_8B], 1, chunk=16 << 20, name="deliver_qwen3_8b_layer"),
    ]


def log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def split(rng, total):
    """total elements as one segment, a layer's tensors, or equal layers, odd sizes among them."""
    how = rng.choice(["one", "one", "tensors", "layers"])
    if how == "one" or total < 4096:
        return [total | (rng.random() < 0.5)], True
    if how == "layers":
        k = rng.randint(2, 32)
        return k * [max(1, total // k)], True
    w = [rng.random() ** 2 + 1e-3 for _ in range(rng.randint(2, 12))]
    return [max(1, int(total * x / sum(w))) for x in w], False


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["noalloc", "norm", "stream", "stream", "route", "deliver"])
    ranks = rng.choice([1, 2, 3, 4, 4, 5, 6, 8, 8, 12, 16])
    outliers = rng.choice([0.0, 0.01])
    sigma = rng.choice([1e-4, 5e-4, 1e-3])
    if kind in ("step", "noalloc", "norm"):
        # at most the bytes of the largest listed call
        top = 42 * QWEN25_72B // (26 + 2 * ranks)
        if kind == "noalloc":
            top = min(top, 512 << 20)
        sizes, flat = split(rng, log_uniform(rng, 20000, top))
        return case(kind, sizes, ranks, flat=flat, sigma=sigma, outliers=outliers,
                    want_norm=kind == "norm" or rng.random() < 0.5)
    ranks = min(ranks, 8)
    total = log_uniform(rng, 2000000, QWEN3_8B * 34 // max(34, 26 + 2 * ranks))
    chunk = TILE * log_uniform(rng, 16, 512)
    if kind == "deliver":
        return case(kind, [total], 1, chunk=chunk)
    sizes, _ = split(rng, total)
    return case(kind, sizes, ranks, sigma=sigma, outliers=outliers, want_norm=True, chunk=chunk,
                bf16=kind == "route" and rng.random() < 0.5)


# ---- inputs ----------------------------------------------------------------

def layout(case):
    """Segment sizes, their offsets in a flat buffer (16-byte aligned for
    every type) and the buffer's length."""
    sizes = [int(x) for x in case["sizes"].split(",")]
    offs, at = [], 0
    for n in sizes:
        offs.append(at)
        at += (n + 63) // 64 * 64
    return sizes, offs, at


def fill(gen, sizes, offs, out, values):
    """out[segment] = values(n) piece by piece; the gaps between segments stay zero."""
    for n, o in zip(sizes, offs):
        for a in range(0, n, PIECE):
            k = min(PIECE, n - a)
            out[o + a:o + a + k] = values(gen, k)


def normal(sigma):
    return lambda gen, n: torch.randn(n, generator=gen, device=DEV).mul_(sigma)


def gradient(case):
    sigma, share = case["sigma"], case["outliers"]

    def values(gen, n):
        x = torch.randn(n, generator=gen, device=DEV).mul_(sigma)
        if share:
            x.mul_(torch.where(torch.rand(n, generator=gen, device=DEV) < share, 100.0, 1.0))
        return x
    return values


def second_moment(case):
    sigma = case["sigma"]
    return lambda gen, n: torch.randn(n, generator=gen, device=DEV).mul_(sigma).square_().add_(1e-3 * sigma * sigma)


def inputs(case, seed, states=True, grads=True):
    """Flat master, first and second moment (mid-training values) and rank gradients on the GPU."""
    sizes, offs, total = layout(case)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))

    def made(values, dtype):
        t = torch.zeros(total, dtype=dtype, device=DEV)
        fill(gen, sizes, offs, t, values)
        return t
    p = m = v = None
    if states:
        p = made(normal(MASTER_SIGMA), torch.float32)
        if case["kind"] != "deliver":
            m = made(normal(0.3 * case["sigma"]), torch.float32)
            v = made(second_moment(case), torch.float32)
    g = [made(gradient(case), torch.bfloat16) for _ in range(case["ranks"])] if grads else []
    return p, m, v, g


class Context:
    """An sdp context that is destroyed with the state that holds it."""

    def __init__(self, **kw):
        self.handle = sdp.sdp_ctx_create(0, **kw)
        weakref.finalize(self, sdp.sdp_ctx_destroy, self.handle)


def pinned(sample):
    """A pinned host array (sdp_host_alloc) with the GPU tensor's contents, as a CPU tensor."""
    bits = np.float32 if sample.dtype == torch.float32 else np.int16
    buf = sdp.HostBuffer(sample.numel() * sample.element_size())
    t = torch.from_numpy(buf.view(bits, sample.numel()))
    if bits is np.int16:
        t = t.view(torch.bfloat16)
    t.copy_(sample)
    return t


def prepare(case, seed):
    kind, R = case["kind"], case["ranks"]
    sizes, offs, total = layout(case)
    st = {"case": case, "hp": sdp.make_params(step=STEP, **HP)}
    if kind == "deliver":
        p = inputs(case, seed, grads=False)[0]
        st["p"] = p.cpu()
        st["window"] = torch.zeros(total, dtype=torch.bfloat16, device=DEV)
        st["ctx"] = Context(max_chunk_elems=case["chunk"], max_ranks=1)
        return st
    p, m, v, g = inputs(case, seed, states=kind != "norm")
    pb = None if kind == "norm" else p.to(torch.bfloat16)
    if kind == "stream":
        p, m, v, pb = (pinned(t) for t in (p, m, v, pb))
        g = [pinned(t) for t in g]
    elif kind == "route":
        p, m, v, pb = (t.cpu() for t in (p, m, v, pb))
    cut = lambda t: [t[o:o + n] for n, o in zip(sizes, offs)]
    if not case["flat"]:
        cut = lambda t: [t[o:o + n].clone() for n, o in zip(sizes, offs)]
    if kind == "norm":
        gs = [cut(t) for t in g]
        st["sets"] = gs
        st["segs"] = sdp.Segments([(0, 0, 0, 0, [gs[r][k].data_ptr() for r in range(R)], n)
                                   for k, n in enumerate(sizes)])
    else:
        ps, ms, vs, pbs, gs = cut(p), cut(m), cut(v), cut(pb), [cut(t) for t in g]
        st["sets"] = (ps, ms, vs, pbs, gs)
        st["segs"] = sdp.segments_from_tensors([(ps[k], ms[k], vs[k], pbs[k], [gs[r][k] for r in range(R)])
                                                for k in range(len(sizes))])
        st["out"] = [p, m, v, pb] if case["flat"] else [ps, ms, vs, pbs]
    if kind in ("step", "norm"):
        st["ctx"] = Context(max_ranks=R)
    elif kind in ("stream", "route"):
        st["ctx"] = Context(max_chunk_elems=case["chunk"], max_ranks=R)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "deliver":
        sdp.sdp_deliver_params(st["ctx"].handle, st["p"].data_ptr(), st["window"].data_ptr(), st["p"].numel(),
                               case["chunk"])
        return st["window"]
    if kind == "stream":
        norm = sdp.sdp_stream_step(st["ctx"].handle, st["segs"], st["hp"], case["chunk"])
        return st["out"] + [norm]
    if kind == "route":
        norm = sdp.sdp_host_update_step(st["ctx"].handle, st["segs"], st["hp"], case["chunk"],
                                        sdp.SDP_GBAR_BF16 if case["bf16"] else sdp.SDP_GBAR_F32)
        return st["out"] + [norm]
    stream = torch.cuda.current_stream()
    if kind == "norm":
        return sdp.sdp_grad_norm(st["ctx"].handle, st["segs"], True, 0, stream)
    if kind == "noalloc":
        norm = sdp.sdp_agg_adam_step_noalloc(st["segs"], st["hp"], stream, case["want_norm"])
    else:
        norm = sdp.sdp_agg_adam_step(st["ctx"].handle, st["segs"], st["hp"], 0, stream, case["want_norm"])
    return st["out"] + [norm] if case["want_norm"] else st["out"]


def work(case):
    """Bytes: each rank gradient and state read once, each state and BF16
    parameter written once.  Operations: the rank sums and their square in the
    norm, and about 20 for AdamW on an element."""
    n = sum(layout(case)[0])
    R = case["ranks"]
    if case["kind"] == "deliver":
        return {"bytes": 6 * n, "flops": 0}
    if case["kind"] == "norm":
        return {"bytes": 2 * R * n, "flops": (R + 3) * n}
    return {"bytes": (2 * R + 26) * n, "flops": (R + 23) * n}


def tolerance(case):
    """A delivery is whole bytes.  A step's states are rounded to 32 bits
    (2.5e-8 away from 64-bit results in the 2-norm); a last-bit difference
    there can turn the BF16 rounding of a parameter next to a tie, and one
    such parameter among the smallest call's 20,000 is 3e-5."""
    if case["kind"] == "deliver":
        return "exact"
    if case["kind"] == "norm":
        return {"rel": 1e-7}
    return {"rel": 4e-5}


def exact(case, seed):
    """The same outputs from plain torch in 64 bits."""
    kind, R = case["kind"], case["ranks"]
    if kind == "deliver":
        return inputs(case, seed, grads=False)[0].double().to(torch.bfloat16)
    sizes, offs, total = layout(case)
    p, m, v, g = inputs(case, seed, states=kind != "norm")

    def mean(a, b):
        s = g[0][a:b].double()
        for t in g[1:]:
            s += t[a:b].double()
        return s / R
    pieces = [(a, min(a + PIECE, total)) for a in range(0, total, PIECE)]
    norm = float(sum(mean(a, b).square().sum() for a, b in pieces).sqrt())
    if kind == "norm":
        return norm
    clip = min(1.0, HP["max_grad_norm"] / (norm + 1e-6))
    b1, b2, lr = HP["beta1"], HP["beta2"], HP["lr"]
    host = kind in ("stream", "route")
    out = [torch.empty(total, dtype=torch.float64, device="cpu" if host else DEV) for _ in range(3)]
    out.append(torch.empty(total, dtype=torch.bfloat16, device="cpu" if host else DEV))
    for a, b in pieces:
        x = mean(a, b)
        if case["bf16"]:
            x = x.float().to(torch.bfloat16).double()
        x *= clip
        pd = p[a:b].double()
        m1 = b1 * m[a:b].double() + (1 - b1) * x
        v1 = b2 * v[a:b].double() + (1 - b2) * x * x
        p1 = pd - lr * HP["weight_decay"] * pd
        p1 -= lr / (1 - b1 ** STEP) * m1 / ((v1 / (1 - b2 ** STEP)).sqrt() + HP["eps"])
        for o, x in zip(out, (p1, m1, v1, p1.to(torch.bfloat16))):
            o[a:b] = x
    if not case["flat"]:
        out = [[t[o:o + n] for n, o in zip(sizes, offs)] for t in out]
    return out + [norm] if case["want_norm"] else out
