"""Short fp32 sequences (rows of up to 128 bytes): the kernels that keep one, two, three or four 16-row
tiles per wave, at the edges of their ranges.  What masked rows hold must not matter: their loads go
nowhere, with one tile per wave by key bytes that do not pass through LDS."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2602_06935_amd import binding
from tests.gpu_util import bar_for, check_tensor, to_f64, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,B,H,N,fmap", [
    (32, 5, 2, 1, "cosine"), (32, 5, 2, 17, "elu1"), (16, 5, 2, 63, "cosine"), (32, 5, 2, 64, "cosine"),   # one
    (32, 5, 2, 65, "cosine"), (16, 5, 2, 128, "elu1"),                                                     # two
    (32, 5, 2, 129, "cosine"), (32, 5, 2, 192, "elu1"),                                                    # three
    (32, 5, 2, 193, "cosine"),                                                                             # four
])
def test_kept_tiles(oracle, d, B, H, N, fmap):
    print(f"[kept tiles] B={B} H={H} N={N} d={d} {fmap}", flush=True)
    rng = np.random.default_rng(5100 + N + d)
    Q, K, V, dO = (rng.standard_normal((B, H, N, d)).astype(np.float32) for _ in range(4))
    mask = (rng.random((B, N)) < 0.5).astype(np.uint8)
    mask[0] = np.arange(N) >= N // 2      # padded at the front
    mask[1] = 0                           # no key at all
    tq, tk, tv, tg = (to_gpu(x, "f32") for x in (Q, K, V, dO))
    tm = torch.from_numpy(mask).cuda()
    dead = (tm == 0)[:, None, :, None].expand_as(tk)
    tk2, tv2 = tk.clone(), tv.clone()
    tk2[dead], tv2[dead] = float("nan"), float("inf")
    opts = dict(scale=0.05, eps=1e-6, feature_map=fmap)
    state = torch.empty(B, H, d, d, device="cuda")
    O = binding.cotten_attn_fwd(tq, tk, tv, tm, saved_state=state, **opts)
    grads = binding.cotten_attn_bwd(tq, tk, tv, tm, tg, **opts)
    kept = binding.cotten_attn_bwd(tq, tk2, tv2, tm, tg, saved_state=state, **opts)
    O2 = binding.cotten_attn_fwd(tq, tk2, tv2, tm, **opts)
    grads2 = binding.cotten_attn_bwd(tq, tk2, tv2, tm, tg, **opts)
    torch.cuda.synchronize()
    assert torch.equal(O, O2) and all(torch.equal(a, c) for a, c in zip(grads, grads2))
    if fmap == "elu1":
        ref = (oracle.elu_fwd(Q, K, V, mask, scale=0.05), *oracle.elu_bwd(Q, K, V, dO, mask, scale=0.05))
    else:
        ref = (oracle.fwd_linear(Q, K, V, mask, scale=0.05, eps=1e-6),
               *oracle.bwd(Q, K, V, dO, mask, scale=0.05, eps=1e-6))
    bar = bar_for("f32")
    for n, g, r in zip(("O", "dQ", "dK", "dV"), (O, *grads), ref):
        check_tensor(n, to_f64(g), r, bar)
    for n, g, r in zip(("dQ", "dK", "dV"), kept, ref[1:]):
        check_tensor(n + " (kept state)", to_f64(g), r, bar)
