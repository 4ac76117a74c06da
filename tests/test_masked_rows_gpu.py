"""dK and dV rows of masked keys are exact zeros whatever the rows that take part hold, infinities and NaN
included, next to valid keys of the same 16 and 32 rows: the causal kernels, and the backward of 16-bit rows of
256 bytes that keeps its rows in registers."""
from __future__ import annotations

import pytest
import torch

from paper_2602_06935_amd import binding

pytestmark = pytest.mark.gpu

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def check(dtype, slices, N, d, **opts):
    print(f"[masked rows] {dtype} slices={slices} N={N} d={d} {opts}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(slices + N + d)
    Q, K, V, dO = (torch.randn(slices, 1, N, d, device="cuda", generator=gen).to(DTYPES[dtype]) for _ in range(4))
    mask = (torch.rand(slices, N, device="cuda", generator=gen) < 0.5).to(torch.uint8)
    mask[1::3, : N // 2] = 0
    dead = (mask == 0)[:, None, :, None].expand_as(K)
    # (columns that different lanes of a row hold: under ELU + 1 a NaN of Q reaches one row of the state only)
    for what, column, value in (("dO", 3, float("inf")), ("Q", 3, float("nan")), ("Q", 11, float("nan")), ("Q", d - 1, float("nan"))):
        x = dict(Q=Q.clone(), dO=dO.clone())
        x[what][:, :, N - 1, column] = value
        for layout in ("bhnd", "bnhd"):
            to = lambda t: t if layout == "bhnd" else t.permute(0, 2, 1, 3).contiguous()
            _, dK, dV = binding.cotten_attn_bwd(to(x["Q"]), to(K), to(V), mask, to(x["dO"]), scale=0.1, eps=1e-6,
                                                layout=layout, **opts)
            for g in (dK, dV):                                  # (of either sign would be equal)
                assert (to(g)[dead].view(torch.int32 if dtype == "f32" else torch.int16) == 0).all(), (what, column, layout)
            assert not torch.isfinite(to(dV).float()).all()     # (it is not for want of anything to hide)


@pytest.mark.parametrize("dtype,slices,N,d", [
    ("bf16", 6, 50, 64), ("f16", 300, 50, 32),                          # four waves; own rows as they are
    ("bf16", 300, 100, 64), ("f16", 6, 200, 64),                        # eight, thirteen
    ("bf16", 6, 300, 64), ("f32", 6, 100, 32), ("f32", 6, 100, 64),     # the walk over chunks
])
def test_causal(dtype, slices, N, d):
    check(dtype, slices, N, d, causal=True)


@pytest.mark.parametrize("fmap", ["cosine", "elu1"])
@pytest.mark.parametrize("dtype,slices,N,d", [
    ("bf16", 300, 50, 128), ("f16", 100, 100, 128), ("bf16", 100, 150, 128), ("f16", 100, 250, 128),   # one to four rounds
])
def test_16bit_wide_kept(dtype, slices, N, d, fmap):
    check(dtype, slices, N, d, feature_map=fmap)
