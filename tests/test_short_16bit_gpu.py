"""Short 16-bit sequences (rows of up to 128 bytes, at most 128 rows): a workgroup of four waves (64 rows)
or eight per slice, at the edges of tiles and ranges, rows of 128, 64 and 32 bytes, both feature maps,
both layouts, per-slice scales with their gradient, the state the forward writes."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2602_06935_amd import binding
from tests.gpu_util import bar_for, check_tensor, rel_l2, to_f64, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,B,H,N,fmap", [
    ("bf16", 64, 5, 2, 9, "cosine"), ("f16", 32, 5, 2, 16, "cosine"), ("bf16", 16, 5, 2, 33, "elu1"),
    ("f16", 64, 5, 2, 64, "elu1"), ("bf16", 32, 150, 2, 64, "cosine"),       # four waves
    ("bf16", 64, 5, 2, 65, "cosine"), ("f16", 16, 5, 2, 112, "cosine"), ("bf16", 32, 5, 2, 113, "elu1"),
    ("f16", 64, 5, 2, 128, "elu1"), ("bf16", 64, 150, 2, 128, "cosine"),     # eight
    ("bf16", 64, 5, 2, 129, "cosine"),                                       # the shortest beyond
])
def test_short_16bit(oracle, dtype, d, B, H, N, fmap):
    print(f"[short 16 bit] {dtype} B={B} H={H} N={N} d={d} {fmap}", flush=True)
    rng = np.random.default_rng(6200 + N + d)
    Q, K, V, dO = (to_gpu(rng.standard_normal((B, H, N, d)).astype(np.float32) * 0.5, dtype) for _ in range(4))
    mask = (rng.random((B, N)) < 0.5).astype(np.uint8)
    mask[0] = np.arange(N) >= N // 2      # padded at the front
    mask[1] = 0                           # no key at all
    mask[2] = 1
    tm = torch.from_numpy(mask).cuda()
    dead = (tm == 0)[:, None, :, None].expand_as(K)
    K2, V2 = K.clone(), V.clone()
    K2[dead], V2[dead] = float("nan"), float("inf")
    ss = torch.rand(B, H, device="cuda") * 0.05 + 0.01
    opts = dict(slice_scale=ss, eps=1e-6, feature_map=fmap)
    state = torch.empty(B, H, d, d, device="cuda")
    dlog = torch.empty(B, H, device="cuda")
    O = binding.cotten_attn_fwd(Q, K, V, tm, saved_state=state, **opts)
    grads = binding.cotten_attn_bwd(Q, K, V, tm, dO, dlog_scale=dlog, **opts)
    sw = lambda t: t.permute(0, 2, 1, 3).contiguous()
    O2 = binding.cotten_attn_fwd(sw(Q), sw(K2), sw(V2), tm, layout="bnhd", **opts)
    grads2 = binding.cotten_attn_bwd(sw(Q), sw(K2), sw(V2), tm, sw(dO), layout="bnhd", saved_state=state, **opts)
    unmasked = binding.cotten_attn_fwd(Q, K, V, None, **opts)
    torch.cuda.synchronize()
    assert torch.equal(sw(O), O2) and all(torch.equal(sw(a), c) for a, c in zip(grads, grads2))
    assert torch.equal(unmasked[2], O[2])
    s64 = ss.double().cpu().numpy()[:, :, None, None]
    q, k, v, g = (to_f64(t) for t in (Q, K, V, dO))
    if fmap == "elu1":
        ref = (oracle.elu_fwd(q, k, v, mask, scale=1.0), *oracle.elu_bwd(q, k, v, g, mask, scale=1.0))
    else:
        ref = (oracle.fwd_linear(q, k, v, mask, scale=1.0, eps=1e-6), *oracle.bwd(q, k, v, g, mask, scale=1.0, eps=1e-6))
    ref = [r * s64 for r in ref]
    bar = bar_for(dtype)
    for n, t, r in zip(("O", "dQ", "dK", "dV"), (O, *grads), ref):
        check_tensor(n, to_f64(t), r, bar)
    # (a sum over all rows of a slice, with cancellation: five times the bar, as elsewhere)
    assert rel_l2(dlog.double().cpu().numpy(), (g * ref[0]).sum((2, 3))) <= 5 * bar
    ref_state = (np.einsum("bn,bhnc,bhne->bhce", mask, np.where(k > 0, k + 1, np.exp(np.minimum(k, 0))), v) if fmap == "elu1"
                 else oracle.state(K.float().cpu().numpy(), V.float().cpu().numpy(), mask))
    assert rel_l2(state.double().cpu().numpy(), ref_state) <= bar


@pytest.mark.parametrize("dtype,d,B,H,N", [
    ("bf16", 64, 5, 2, 64), ("bf16", 32, 150, 2, 50), ("f16", 64, 260, 1, 64),   # four waves; rows as they are
    ("f16", 16, 5, 2, 65), ("bf16", 64, 150, 2, 128), ("bf16", 64, 5, 2, 129),   # eight, thirteen
])
def test_short_causal_16bit(oracle, dtype, d, B, H, N):
    print(f"[short 16 bit, causal] {dtype} B={B} H={H} N={N} d={d}", flush=True)
    rng = np.random.default_rng(6900 + N + d)
    x = [rng.standard_normal((B, H, N, d)).astype(np.float32) * 0.5 for _ in range(4)]
    for t in x[:2]:                       # long and short rows of Q and K
        t[rng.random((B, H, N)) < 0.05] *= 300.0
        t[rng.random((B, H, N)) < 0.05] *= 1e-3
    Q, K, V, dO = (to_gpu(t, dtype) for t in x)
    mask = (rng.random((B, N)) < 0.7).astype(np.uint8)
    mask[:, 0] = 1
    mask[1] = 0                           # no key at all
    tm = torch.from_numpy(mask).cuda()
    dead = (tm == 0)[:, None, :, None].expand_as(K)
    K2, V2 = K.clone(), V.clone()
    K2[dead], V2[dead] = float("nan"), float("inf")
    opts = dict(scale=0.05, eps=1e-6, causal=True)
    O = binding.cotten_attn_fwd(Q, K, V, tm, **opts)
    grads = binding.cotten_attn_bwd(Q, K, V, tm, dO, **opts)
    sw = lambda t: t.permute(0, 2, 1, 3).contiguous()
    O2 = binding.cotten_attn_fwd(sw(Q), sw(K2), sw(V2), tm, layout="bnhd", **opts)
    grads2 = binding.cotten_attn_bwd(sw(Q), sw(K2), sw(V2), tm, sw(dO), layout="bnhd", **opts)
    torch.cuda.synchronize()
    assert torch.equal(sw(O), O2) and all(torch.equal(sw(a), c) for a, c in zip(grads, grads2))
    q, k, v, g = (to_f64(t) for t in (Q, K, V, dO))
    ref = (oracle.causal_fwd(q, k, v, mask, scale=0.05, eps=1e-6),
           *oracle.causal_bwd(q, k, v, g, mask, scale=0.05, eps=1e-6))
    for n, t, r in zip(("O", "dQ", "dK", "dV"), (O, *grads), ref):
        assert rel_l2(to_f64(t), r) <= bar_for(dtype), n
    assert all(np.all(to_f64(t)[dead.cpu().numpy()] == 0.0) for t in grads[1:])


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_short_causal_backward_from_rows_as_they_are(oracle, dtype):
    """More than 256 slices of up to 64 rows: dV takes the keys as they are and divides its result, fewer round them after the
    division.  The same sequences one way and the other, both against 64 bits: a rounding less shows (2.9e-3 and 3.3e-3 in bf16)."""
    B, N, d = 300, 50, 64
    print(f"[short 16 bit, causal] rows as they are, {dtype}", flush=True)
    rng = np.random.default_rng(6500)
    Q, K, V, dO = (to_gpu(rng.standard_normal((B, 1, N, d)).astype(np.float32), dtype) for _ in range(4))
    opts = dict(scale=0.05, eps=1e-6, causal=True)
    raw = binding.cotten_attn_bwd(Q, K, V, None, dO, **opts)[2][:256]
    few = binding.cotten_attn_bwd(Q[:256], K[:256], V[:256], None, dO[:256], **opts)[2]
    ref = oracle.causal_bwd(*(to_f64(t[:256]) for t in (Q, K, V, dO)), np.ones((256, N), np.uint8), scale=0.05, eps=1e-6)[2]
    e_raw, e_few = rel_l2(to_f64(raw), ref), rel_l2(to_f64(few), ref)
    print(f"[short 16 bit, causal]   dV {e_raw:.3e}, rounded {e_few:.3e}", flush=True)
    assert e_raw <= 0.95 * e_few <= bar_for(dtype)


@pytest.mark.parametrize("slices,N,backward", [(1 << 24, 1, True), (1 << 23, 65, False)])
def test_more_slices_than_a_launch_of_one_workgroup_each_admits(oracle, slices, N, backward):
    """Every count up to the 2^24 slices that the entry points take runs: 2^24 workgroups of four waves, or 2^23 of eight,
    would be 2^32 threads, which no launch has."""
    d, H = 16, 8
    print(f"[short 16 bit] {slices} slices x {N} rows", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(slices + N)
    make = lambda: torch.empty(slices // H, H, N, d, device="cuda", dtype=torch.bfloat16).normal_(generator=gen)
    Q = make()
    K, V, dO = (make(), make(), make()) if N == 1 else (Q, Q, Q)     # (17 GB each at 65 rows)
    opts = dict(scale=0.5, eps=1e-6)
    out = [binding.cotten_attn_fwd(Q, K, V, None, **opts)]
    if backward:
        out += binding.cotten_attn_bwd(Q, K, V, None, dO, **opts)
    few = torch.tensor([0, 1, slices // H // 2, slices // H - 1], device="cuda")
    q, k, v, g = (to_f64(t[few]) for t in (Q, K, V, dO))
    mask = np.ones((len(few), N), np.uint8)
    ref = (oracle.fwd_linear(q, k, v, mask, **opts), *oracle.bwd(q, k, v, g, mask, **opts))
    bar = bar_for("bf16")
    for n, t, r in zip(("O", "dQ", "dK", "dV"), out, ref):
        check_tensor(n, to_f64(t[few]), r, bar)
    del Q, K, V, dO, out, t
    torch.cuda.empty_cache()
