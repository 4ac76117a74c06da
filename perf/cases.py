"""The calls that this library is timed on: training steps and forwards of one attention layer, over
the sizes, element types and options of the paper's sweeps, `inputs.WORKLOADS`, the tests and the
benchmark (sequence lengths 20 ... 4096, embeddings 64 ... 256 with two to four heads, left-padded
histories).

A case is a dict of
    B, H, N, d       sizes; `dtype` "f32", "bf16" or "f16"
    direction        "forward" (serving) or "train" (forward and backward)
    via              how the program calls the library: "call" the binding's functions, "autograd"
                     `cosine_attention` and `torch.autograd.grad`, "graph" the same binding calls
                     captured once into a HIP graph that is replayed for every step (what a loop of
                     short steps over fixed buffers does, and what `bench.py` does)
    layout           "bhnd" or "bnhd"
    lengths          "full" (no mask), "uniform" (5 ... N valid keys per sequence; from a quarter of N
                     on for long histories) or "geometric" (mean 0.6 N)
    causal, elu1     the variant with the causal mask; the ELU + 1 map in place of the L2 norms
    keep_state       the forward keeps the d x d states for its backward
    normaliser       the learnable normaliser: scales n_b^(-m_h) made before the forward, their
                     gradient carried back to m
"""
import math

import torch

from paper_2602_06935_amd import binding
from paper_2602_06935_amd.autograd import cosine_attention

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
ELEM_BYTES = {"f32": 4, "bf16": 2, "f16": 2}
EPS = 1e-6
TINY_ROWS = 0.01          # share of the rows of Q and of K that are next to zero
LARGEST_TENSOR = 1024 * 4 * 200 * 64 * 2    # bytes of one tensor of the largest listed case
SMALLEST_TENSOR = 4 * 2 * 50 * 32 * 4       # and of the smallest


def _case(name, B, H, N, d, dtype, direction="train", via="call", layout="bhnd", lengths="uniform",
          causal=False, elu1=False, keep_state=False, normaliser=False):
    c = dict(B=B, H=H, N=N, d=d, dtype=dtype, direction=direction, via=via, layout=layout,
             lengths=lengths, causal=causal, elu1=elu1, keep_state=keep_state, normaliser=normaliser)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one small request served in fp32 (configuration 1): latency of a single call
        _case("serve_small_f32", 4, 2, 50, 32, "f32", "forward", lengths="full"),
        # short histories in fp32 (configuration 2): the step is launch-bound, so its loop is a graph
        _case("train_n50_f32", 256, 2, 50, 32, "f32", via="graph"),
        # the paper's N = 200 point in fp32, embedding 64 (configuration 3), state kept
        _case("train_n200_f32", 256, 2, 200, 32, "f32", via="graph", lengths="geometric",
              keep_state=True),
        # embedding 256 with four heads under bf16 mixed precision (configuration 4) at a large
        # batch, inside a model: autograd, tensors as the projections around the layer leave them
        _case("train_n200_bf16", 1024, 4, 200, 64, "bf16", via="autograd", layout="bnhd"),
        # long histories (configuration 5), state kept
        _case("train_long_bf16", 16, 4, 4096, 64, "bf16", keep_state=True),
        # embedding 256 with two heads, bf16, learnable normaliser
        _case("train_emb256_bf16", 512, 2, 200, 128, "bf16", normaliser=True),
        # the same embedding without mixed precision
        _case("train_emb256_f32", 256, 2, 200, 128, "f32"),
        # embedding 128 without mixed precision, N = 100, inside a model
        _case("train_emb128_f32", 512, 2, 100, 64, "f32", via="autograd", layout="bnhd"),
        # serving long histories, embedding 256 with two heads
        _case("serve_long_bf16", 16, 2, 3000, 128, "bf16", "forward"),
        # causal variant: histories of a thousand items, bf16, ragged last tile
        _case("causal_n1001_bf16", 64, 4, 1001, 64, "bf16", causal=True),
        # causal variant at embedding 128 in fp32
        _case("causal_n200_f32", 64, 2, 200, 64, "f32", causal=True),
        # the linear-attention comparison model (ELU + 1), fp16, odd length
        _case("elu1_n197_f16", 256, 4, 197, 64, "f16", layout="bnhd", elu1=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        dtype = rng.choice(["f32", "bf16", "bf16", "f16"])
        d = rng.choice([32, 64, 128] if dtype == "f32" else [32, 64, 64, 128])
        H = rng.choice([1, 2, 2, 4, 8])
        N = _log_int(rng, 20, 4096)
        B = _log_int(rng, 1, 1024)
        size = B * H * N * d * ELEM_BYTES[dtype]
        if not SMALLEST_TENSOR <= size <= LARGEST_TENSOR:
            continue
        kind = rng.choice(["cosine"] * 6 + ["causal", "causal", "elu1"])
        causal, elu1 = kind == "causal" and d <= 64, kind == "elu1"
        plain = not causal and not elu1
        direction = rng.choice(["train", "train", "forward"])
        via = rng.choice(["call", "call", "autograd", "graph"])
        if via == "autograd" and (direction == "forward" or not plain):
            via = "call"
        keep_state = plain and via != "autograd" and direction == "train" and rng.random() < 0.4
        normaliser = plain and via != "autograd" and rng.random() < 0.2
        return _case(None, B, H, N, d, dtype, direction, via, rng.choice(["bhnd", "bnhd"]),
                     rng.choice(["uniform", "uniform", "geometric", "full"]), causal, elu1,
                     keep_state, normaliser)


def _length_range(N):
    lo = min(N, 5 if N <= 512 else N // 4)
    return lo, N


def _valid_fraction(case):
    """Expected share of valid keys."""
    N, kind = case["N"], case["lengths"]
    if kind == "full":
        return 1.0
    lo, hi = _length_range(N)
    if kind == "uniform":
        return (lo + hi) / 2 / N
    # clip(Geom(p), lo, hi): lo + sum over j = lo ... hi-1 of P(length > j)
    q = 1.0 - min(1.0, 1.0 / (0.6 * N))
    return (lo + sum(q ** j for j in range(lo, hi))) / N


def work(case):
    """Each input read once and each output written once: rows of Q, dO and of every result whole, rows
    of K and V where the key is valid.  Flops of the linear form (states and their products)."""
    B, H, N, d = case["B"], case["H"], case["N"], case["d"]
    f, tensor = _valid_fraction(case), B * H * N * d * ELEM_BYTES[case["dtype"]]
    n_bytes, flops = (2 + 2 * f) * tensor, (2 + 2 * f) * d * d * B * H * N
    if case["lengths"] != "full":
        n_bytes += B * N
    if case["direction"] == "train":
        n_bytes += (5 + 2 * f) * tensor + (B * N if case["lengths"] != "full" else 0)
        flops += (4 + (4 if case["keep_state"] else 6) * f) * d * d * B * H * N
    if case["keep_state"]:
        n_bytes += 2 * B * H * d * d * 4
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    """About four times the distance from an fp64 evaluation (measured: 1.5e-7 ... 3.4e-7 in fp32, 2.9e-3
    ... 3.3e-3 in bf16 and an eighth of that in fp16, where outputs, unit rows and state operands are
    rounded to 16 bits).  Single values that come out small by cancellation are further off."""
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 1e-4}
    return {"rel": 1.2e-2, "max": 0.4} if case["dtype"] == "bf16" else {"rel": 1.6e-3, "max": 0.05}


class _State:
    """What the program holds: inputs, and with "graph" the captured step and its result buffers."""


def _lengths(case, gen, device):
    B, N, kind = case["B"], case["N"], case["lengths"]
    if kind == "full":
        return None
    lo, hi = _length_range(N)
    u = torch.rand(B, generator=gen, device=device, dtype=torch.float64)
    if kind == "uniform":
        return (lo + torch.floor(u * (hi - lo + 1))).clamp(lo, hi).to(torch.int32)
    p = min(1.0, 1.0 / (0.6 * N))
    length = torch.full_like(u, 1.0) if p >= 1.0 else torch.ceil(torch.log1p(-u) / math.log1p(-p))
    return length.clamp(lo, hi).to(torch.int32)


def prepare(case, seed):
    device = torch.device("cuda", torch.cuda.current_device())
    gen = torch.Generator(device=device)
    gen.manual_seed(int(seed))
    B, H, N, d, dtype = case["B"], case["H"], case["N"], case["d"], DTYPES[case["dtype"]]
    shape = (B, H, N, d) if case["layout"] == "bhnd" else (B, N, H, d)
    sigma = 1.0 if case["dtype"] == "f32" else 0.5

    def normal(scale, tiny):
        x = torch.randn(shape, generator=gen, device=device) * scale
        if tiny:
            rows = torch.rand(shape[:3], generator=gen, device=device) < TINY_ROWS
            x *= torch.where(rows, 1e-4, 1.0).unsqueeze(-1)
        return x.to(dtype)

    s = _State()
    s.case = dict(case)
    s.q, s.k, s.v = normal(sigma, True), normal(sigma, True), normal(sigma, False)
    train = case["direction"] == "train"
    s.dO = normal(1.0, False) if train else None
    lengths = _lengths(case, gen, device)
    s.mask = None
    if lengths is not None:   # histories are padded on the left
        s.mask = (torch.arange(N, device=device)[None, :] >= (N - lengths)[:, None]).to(torch.uint8)
    s.n = lengths
    s.m = torch.rand(H, generator=gen, device=device) * 0.5 + 0.5 if case["normaliser"] else None
    s.kept = torch.empty(B, H, d, d, device=device) if case["keep_state"] else None
    s.graph = s.results = None
    if case["via"] == "autograd":
        for t in (s.q, s.k, s.v):
            t.requires_grad_(True)
    elif case["via"] == "graph":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _calls(s)
        torch.cuda.current_stream().wait_stream(side)
        s.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s.graph):
            s.results = _calls(s)
    return s


def _calls(s):
    c = s.case
    B, H, N = c["B"], c["H"], c["N"]
    opts = dict(eps=EPS, layout=c["layout"], causal=c["causal"],
                feature_map="elu1" if c["elu1"] else "cosine")
    scales = None
    if s.kept is not None:
        opts["saved_state"] = s.kept
    if s.m is not None:
        scales = binding.cotten_normaliser_fwd(s.m, s.n, B, N)
        opts["slice_scale"] = scales
    else:
        opts["scale"] = 1.0 / N
    out = {"O": binding.cotten_attn_fwd(s.q, s.k, s.v, s.mask, **opts)}
    if scales is not None:
        out["scales"] = scales
    if s.kept is not None:
        out["state"] = s.kept
    if s.dO is None:
        return out
    if scales is not None:
        opts["dlog_scale"] = torch.empty_like(scales)
    out["dQ"], out["dK"], out["dV"] = binding.cotten_attn_bwd(s.q, s.k, s.v, s.mask, s.dO, **opts)
    if scales is not None:
        out["dlog"] = opts["dlog_scale"]
        out["dm"] = binding.cotten_normaliser_bwd(opts["dlog_scale"], s.n, N)
    return out


def run(state):
    if state.graph is not None:
        state.graph.replay()
        return state.results
    if state.case["via"] == "autograd":
        O = cosine_attention(state.q, state.k, state.v, state.mask, scale=1.0 / state.case["N"],
                             eps=EPS, layout=state.case["layout"])
        dQ, dK, dV = torch.autograd.grad(O, (state.q, state.k, state.v), state.dO)
        return {"O": O, "dQ": dQ, "dK": dK, "dV": dV}
    return _calls(state)
