"""fp32 rows as three bf16 pieces on the matrix cores: parity against the fp64 oracle where the
kernels for 256- and 512-byte rows change shape - one row, ends of tiles (16), of the rounds of the
state walk (64), more tiles than waves (4 and 8), slices in groups of eight, sequences cut over
several workgroups - with values over many powers of two.

Bound per slice 1e-6: a product of two values as six products of their pieces is within 2^-22 (2.4e-7) of it
at worst (each value cut to 8 bits, then rounded to 8 more: the first remainder is below 2^-7 of the value, the
second below 2^-16), and the fp32 sums that follow (N, then d_h terms, then one rounding per result) add a
few units of 2^-24 on random inputs; a missing or misplaced piece would show as 2^-16 or more."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2602_06935_amd import binding
from tests.gpu_util import FP32_BAR, check_tensor, rel_l2, to_f64, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,N,d", [
    (3, 1, 1, 64), (2, 2, 16, 64), (3, 3, 65, 64), (1, 2, 257, 64), (9, 1, 130, 32), (2, 1, 700, 64),
    (3, 1, 1, 128), (2, 2, 17, 128), (3, 3, 64, 128), (1, 1, 129, 128), (2, 2, 255, 128), (3, 1, 257, 128),
    (2, 1, 700, 128), (130, 2, 300, 128),
])
@pytest.mark.parametrize("feature_map", ["cosine", "elu1"])
def test_fp32_pieces(oracle, B, H, N, d, feature_map):
    if feature_map == "elu1" and B > 100:
        pytest.skip("one map is enough at this size")
    print(f"[fp32 pieces] B={B} H={H} N={N} d={d} {feature_map}", flush=True)
    rng = np.random.default_rng(9100 + N + d + B)
    Q, K, V, dO = (rng.standard_normal((B, H, N, d)).astype(np.float32) for _ in range(4))
    if feature_map == "cosine":
        for x in (Q, K):                     # the map takes the scale of a row out again
            x *= np.exp2(rng.integers(-8, 9, (B, H, N, 1))).astype(np.float32)
        if B * H < 20:                       # (larger cases are held tensor by tensor)
            V *= np.exp2(rng.integers(-30, 31, (B, H, 1, 1))).astype(np.float32)
    mask = (np.arange(N)[None, :] >= rng.integers(0, N, B)[:, None]).astype(np.uint8)
    if B > 1:
        mask[1] = rng.random(N) < 0.5
        mask[1, N // 2] = 1
    if B > 2:
        mask[2] = 0
    tq, tk, tv, tg = (to_gpu(x, "f32") for x in (Q, K, V, dO))
    tm = torch.from_numpy(mask).cuda()
    opts = dict(scale=0.25, eps=1e-6, feature_map=feature_map)
    dlog = torch.zeros(B, H, device="cuda")
    O = binding.cotten_attn_fwd(tq, tk, tv, tm, **opts)
    grads = binding.cotten_attn_bwd(tq, tk, tv, tm, tg, dlog_scale=dlog, **opts)
    again = binding.cotten_attn_bwd(tq, tk, tv, tm, tg, **opts)
    torch.cuda.synchronize()
    if feature_map == "cosine":
        ref_o = oracle.fwd_linear(Q, K, V, mask, scale=0.25, eps=1e-6)
        refs = oracle.bwd(Q, K, V, dO, mask, scale=0.25, eps=1e-6)
    else:
        ref_o = oracle.elu_fwd(Q, K, V, mask, scale=0.25)
        refs = oracle.elu_bwd(Q, K, V, dO, mask, scale=0.25)
    assert all(torch.equal(a, b) for a, b in zip(grads, again))
    for name, got, ref in zip(("O", "dQ", "dK", "dV"), (O, *grads), (ref_o, *refs)):
        if B * H >= 20:
            check_tensor(name, to_f64(got), ref, FP32_BAR)
        else:
            for b in range(B):               # V differs by powers of two between slices
                for h in range(H):
                    g, r = to_f64(got)[b, h], ref[b, h]
                    if not r.any():          # no valid key
                        assert not g.any(), (name, b, h)
                        continue
                    e = rel_l2(g, r)
                    # a slice with one key or one row may consist of a cosine near zero
                    assert e <= (1e-6 if N >= 16 and mask[b].sum() > 8 else FP32_BAR), (name, b, h, e)
        dead = np.broadcast_to((mask == 0)[:, None, :, None], ref.shape)
        if name in ("dK", "dV"):
            assert np.all(to_f64(got)[dead] == 0.0)
    ref_dlog = (dO.astype(np.float64) * ref_o).sum(axis=(2, 3))
    size = np.sqrt(((dO.astype(np.float64) * ref_o) ** 2).sum(axis=(2, 3)))  # sums with cancellation
    assert np.all(np.abs(dlog.double().cpu().numpy() - ref_dlog) <= 1e-5 * np.maximum(size, np.abs(ref_dlog)))
