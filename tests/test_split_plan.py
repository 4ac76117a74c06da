"""Where sequences are cut, and into how many workgroups: the rule on the host (through the workspace a call asks for:
one state per slice and workgroup, two in the backward, none where a call is one launch; wide rows that are cut: one
more), and parity on both sides of its lines."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from paper_2602_06935_amd import binding
from tests.gpu_util import bar_for, check_tensor, rel_l2, to_f64, to_gpu

F32, BF16, F16 = binding.COTTEN_F32, binding.COTTEN_BF16, binding.COTTEN_F16


def _splits(slices, N, dtype, bwd):
    side = 32 if dtype == F32 else 64
    need = binding.cotten_attn_workspace_bytes(slices, 1, N, side, dtype, bwd)
    states = need // (slices * side * side * 4 * (2 if bwd else 1))
    assert states * slices * side * side * 4 * (2 if bwd else 1) == need
    return states


@pytest.mark.parametrize("slices,N,dtype,splits", [
    # 16 bits: whole from N / 5 - 10 slices on, at most 170 of them
    (39, 250, BF16, 0), (53, 320, BF16, 3), (54, 320, BF16, 0), (109, 600, F16, 4), (110, 600, F16, 0),
    (169, 2048, BF16, 2), (170, 2048, BF16, 0), (170, 2049, BF16, 2),
    # a workgroup per compute unit of the XCD, no more than sqrt(N / 7) (or ten), blocks of 64 rows
    (1, 300, BF16, 5), (8, 600, BF16, 10), (8, 1500, BF16, 12), (8, 4096, BF16, 22), (9, 4096, BF16, 16),
    (24, 4096, BF16, 10), (32, 2000, F16, 8), (64, 2000, BF16, 4),
    # two where a workgroup would have more than 600 rows, or there are more than eight slices per XCD
    (64, 4096, BF16, 8), (72, 4096, BF16, 7), (100, 2500, BF16, 4), (128, 4096, F16, 4),
    # fp32: two, or three where these fill it better
    (7, 4096, F32, 32), (16, 4096, F32, 16), (64, 4096, F32, 8), (96, 4096, F32, 8), (180, 4096, F32, 4),
    (200, 4096, F32, 2), (119, 320, F32, 3), (120, 320, F32, 0), (128, 321, F32, 3), (168, 470, F32, 3), (169, 470, F32, 0), (255, 864, F32, 2),
])
def test_split_rule(slices, N, dtype, splits):
    assert _splits(slices, N, dtype, True) == splits
    assert _splits(slices, N, dtype, False) == splits


@pytest.mark.parametrize("slices,N,d,fwd,bwd", [
    # forward: a workgroup per compute unit; backward: as many as three roles leave room for, 256 or 384 in all
    (1, 256, 128, 1, 1), (1, 257, 128, 5, 5), (4, 1000, 128, 16, 16), (10, 3500, 128, 19, 8), (20, 1800, 128, 10, 4), (32, 901, 128, 8, 4), (64, 300, 128, 3, 1),
    (46, 300, 128, 5, 1), (46, 301, 128, 5, 2), (46, 1101, 128, 5, 5), (56, 301, 128, 3, 2), (57, 450, 128, 4, 1), (36, 2400, 128, 7, 3), (36, 2401, 128, 7, 7),
    (72, 1000, 128, 3, 1), (72, 1001, 128, 3, 3), (92, 2000, 128, 2, 1), (92, 2401, 128, 5, 5), (103, 4000, 128, 2, 1),
    (129, 700, 128, 1, 1), (129, 701, 128, 1, 3), (170, 1400, 128, 1, 3), (170, 1401, 128, 3, 3), (171, 1401, 128, 1, 3), (193, 4000, 128, 1, 1),
    (64, 1800, 128, 4, 2), (86, 331, 128, 2, 1), (128, 330, 128, 1, 1), (128, 2000, 128, 2, 1), (129, 256, 128, 1, 1), (255, 4000, 128, 1, 1),
    # two pieces per row: up to three workgroups per compute unit
    (1, 3500, 64, 28, 28), (20, 1000, 64, 8, 4), (32, 1000, 64, 8, 8), (64, 328, 64, 1, 1), (64, 420, 64, 4, 1), (64, 1800, 64, 4, 4), (90, 3500, 64, 8, 8),
    (153, 800, 64, 4, 1), (154, 1150, 64, 1, 1), (154, 1151, 64, 4, 1), (192, 1150, 64, 1, 1), (226, 1150, 64, 1, 1), (226, 1151, 64, 3, 1),
    (129, 600, 64, 1, 1), (129, 601, 64, 1, 2), (150, 1000, 64, 4, 2), (151, 1000, 64, 4, 1),
    (128, 1000, 64, 2, 1), (150, 1800, 64, 5, 5), (200, 1600, 64, 3, 1), (250, 1200, 64, 1, 1),
])
def test_wide_fp32_split_rule(slices, N, d, fwd, bwd):
    for is_bwd, parts in ((False, fwd), (True, bwd)):
        need = binding.cotten_attn_workspace_bytes(slices, 1, N, d, F32, is_bwd)
        states = 0 if parts == 1 else (parts + 1) * (2 if is_bwd else 1)
        assert need == slices * states * d * d * 4, (is_bwd, need / (slices * d * d * 4))


# fp32 shapes that are cut in both directions, and a number of parts that they also run in: (d, slices, N, fewest, parts)
FEWER_PARTS = [(128, 4, 700, 2, 3), (64, 1, 1100, 2, 5), (128, 12, 600, 2, 3), (64, 8, 1000, 2, 4), (32, 81, 453, 2, 4), (16, 81, 453, 2, 3),
               (32, 129, 4100, 3, 4)]
# shapes that are cut where there is a workspace and run whole without one: (d, slices, N, fwd, bwd)
WHOLE_WITHOUT = [(128, 129, 1401, 3, 3), (128, 192, 1457, 1, 3), (128, 170, 1401, 3, 3), (64, 129, 601, 1, 2), (32, 168, 321, 3, 3), (16, 168, 440, 3, 3)]


def _bytes(d, slices, parts, is_bwd):
    side, states = (32, parts) if d <= 32 else (d, parts + 1)
    return slices * states * side * side * 4 * (2 if is_bwd else 1)


@pytest.mark.parametrize("d,slices,N,fewest,parts", FEWER_PARTS)
def test_fp32_workspace_smaller_than_asked_for(d, slices, N, fewest, parts):
    """Refused, on the host, below the states of two parts (of rows of 128 bytes: of parts of 2048 rows), and without one."""
    lib = binding.load_library()
    ptrs = (0x1000, 0x2000, 0x3000, None, 0x4000, 0x5000, 0x6000, 0x7000)
    for is_bwd in (False, True):
        for space, size in ((0x10000, _bytes(d, slices, fewest, is_bwd) - 4), (None, 0)):
            p = binding.CottenParams(F32, 0.0, -1.0, space, size)
            if is_bwd:
                assert lib.cotten_attn_bwd_ex(*ptrs, slices, 1, N, d, None, ctypes.byref(p)) == -6
            else:
                assert lib.cotten_attn_fwd_ex(*ptrs[:5], slices, 1, N, d, None, ctypes.byref(p)) == -6


@pytest.mark.gpu
@pytest.mark.parametrize("d,slices,N,fewest,parts", FEWER_PARTS)
def test_fp32_runs_in_fewer_parts(oracle, d, slices, N, fewest, parts):
    """What was refused above runs from that size on, and writes nothing behind it."""
    for n in (fewest, parts):
        print(f"[split plan] fewer parts d={d} {slices} x {N} in {n}", flush=True)
        sizes = [_bytes(d, slices, n, is_bwd) for is_bwd in (False, True)]
        assert all(binding.cotten_attn_workspace_bytes(slices, 1, N, d, F32, x) > sizes[x] for x in (False, True))
        _parity_in(oracle, d, slices, N, sizes)


@pytest.mark.gpu
@pytest.mark.parametrize("d,slices,N,fwd,bwd", WHOLE_WITHOUT)
def test_fp32_runs_whole_without_a_workspace(oracle, d, slices, N, fwd, bwd):
    print(f"[split plan] whole d={d} {slices} x {N}", flush=True)
    for is_bwd, parts in ((False, fwd), (True, bwd)):
        asked = binding.cotten_attn_workspace_bytes(slices, 1, N, d, F32, is_bwd)
        assert asked == (0 if parts == 1 else _bytes(d, slices, parts, is_bwd))
    _parity_in(oracle, d, slices, N, (16, 16))
    # the static scratch serves as a workspace of its size
    q, k, v, g = (torch.randn(slices, 1, N, d, device="cuda") for _ in range(4))
    out = [torch.empty_like(q) for _ in range(3)]
    binding.cotten_attn_bwd(q, k, v, None, g, *out, static_scratch=True)
    ref = binding.cotten_attn_bwd(q, k, v, None, g, workspace=torch.empty(32 << 20, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(out, ref))


def _parity_in(oracle, d, slices, N, sizes):
    tail = 4096
    whole = [torch.full((b + tail,), 0xA5, dtype=torch.uint8, device="cuda") for b in sizes]
    _parity(oracle, "f32", d, slices, N, [w[:b] for w, b in zip(whole, sizes)])
    assert all((w[b:] == 0xA5).all() for w, b in zip(whole, sizes))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d,slices,N", [
    ("f32", 128, 4, 257), ("f32", 128, 86, 340), ("f32", 128, 150, 290), ("f32", 128, 46, 310), ("f32", 128, 72, 1001), ("f32", 128, 92, 2420), ("f32", 128, 131, 1450), ("f32", 64, 20, 333), ("f32", 64, 64, 421),
    ("f32", 64, 150, 1300), ("f32", 64, 131, 650), ("f32", 64, 154, 1150), ("f32", 64, 154, 1151), ("f32", 64, 200, 310), ("bf16", 128, 64, 300), ("bf16", 128, 40, 310), ("f16", 128, 128, 520), ("bf16", 128, 48, 700),
    ("bf16", 128, 32, 1300), ("f16", 128, 150, 1300),
])
def test_wide_rows_on_both_sides_of_the_split_rule(oracle, dtype, d, slices, N):
    print(f"[split plan] {dtype} d={d} {slices} x {N}", flush=True)
    _parity(oracle, dtype, d, slices, N)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,slices,N", [
    ("bf16", 53, 320), ("bf16", 54, 320), ("f16", 170, 1029), ("bf16", 169, 1029), ("bf16", 9, 1531), ("f16", 3, 2300),
    ("f32", 120, 320), ("f32", 168, 321), ("f32", 96, 1100), ("f32", 7, 2049),
])
def test_both_sides_of_the_split_rule(oracle, dtype, slices, N):
    print(f"[split plan] {dtype} {slices} x {N}", flush=True)
    _parity(oracle, dtype, 32 if dtype == "f32" else 64, slices, N)


@pytest.mark.gpu
@pytest.mark.parametrize("d,slices,N", [(128, 129, 1401), (128, 72, 1010), (64, 131, 650), (64, 160, 1100), (32, 150, 400)])
def test_options_where_the_rule_cuts(oracle, d, slices, N):
    """Kept state, d loss / d log(scale), ELU + 1, and a captured call replayed three times, in fp32."""
    print(f"[split plan] options d={d} {slices} x {N}", flush=True)
    rng = np.random.default_rng(91 + N)
    Q, K, V, dO = (rng.standard_normal((slices, 1, N, d)).astype(np.float32) for _ in range(4))
    mask = (np.arange(N)[None, :] >= rng.integers(0, N, slices)[:, None]).astype(np.uint8)
    q, k, v, g = (to_gpu(x, "f32") for x in (Q, K, V, dO))
    m = torch.from_numpy(mask).cuda()
    state, dlog = torch.zeros(slices, 1, d, d, device="cuda"), torch.zeros(slices, 1, device="cuda")
    O = binding.cotten_attn_fwd(q, k, v, m, saved_state=state)
    grads = binding.cotten_attn_bwd(q, k, v, m, g, dlog_scale=dlog)
    kept = binding.cotten_attn_bwd(q, k, v, m, g, saved_state=state)
    elu = (binding.cotten_attn_fwd(q, k, v, m, feature_map="elu1"), *binding.cotten_attn_bwd(q, k, v, m, g, feature_map="elu1"))
    torch.cuda.synchronize()
    bar = bar_for("f32")
    ref_o, refs = oracle.fwd_linear(Q, K, V, mask), oracle.bwd(Q, K, V, dO, mask)
    assert rel_l2(state.double().cpu().numpy(), oracle.state(K, V, mask)) <= bar
    for name, got, ref in zip(("O", "dQ", "dK", "dV", "dQ", "dK", "dV"), (O, *grads, *kept), (ref_o, *refs, *refs)):
        check_tensor(name, to_f64(got), ref, bar)
    few = [np.ascontiguousarray(x[-4:]) for x in (Q, K, V, dO)]  # (that oracle works from the N x N definition)
    for name, got, ref in zip(("O", "dQ", "dK", "dV"), elu, (oracle.elu_fwd(*few[:3], mask[-4:].copy()), *oracle.elu_bwd(*few, mask[-4:].copy()))):
        check_tensor(name, to_f64(got[-4:]), ref, bar)
    ref_dlog = (dO.astype(np.float64) * ref_o).sum(axis=(2, 3))
    size = np.sqrt(((dO.astype(np.float64) * ref_o) ** 2).sum(axis=(2, 3)))  # a sum with cancellation
    assert np.all(np.abs(dlog.double().cpu().numpy() - ref_dlog) <= bar * np.maximum(size, np.abs(ref_dlog)))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        again = (binding.cotten_attn_fwd(q, k, v, m), *binding.cotten_attn_bwd(q, k, v, m, g))
    for _ in range(3):
        for t in again:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(again, (O, *grads)))


def _parity(oracle, dtype, d, slices, N, workspaces=(None, None)):
    rng = np.random.default_rng(3000 + N + slices)
    Q, K, V, dO = (to_f64(to_gpu(rng.standard_normal((slices, 1, N, d)), dtype)).astype(np.float32) for _ in range(4))
    mask = (np.arange(N)[None, :] >= rng.integers(0, N, slices)[:, None]).astype(np.uint8)
    tq, tk, tv, tg = (to_gpu(x, dtype) for x in (Q, K, V, dO))
    tm = torch.from_numpy(mask).cuda()
    O = binding.cotten_attn_fwd(tq, tk, tv, tm, workspace=workspaces[0])
    grads = binding.cotten_attn_bwd(tq, tk, tv, tm, tg, workspace=workspaces[1])
    torch.cuda.synchronize()
    refs = (oracle.fwd_linear(Q, K, V, mask), *oracle.bwd(Q, K, V, dO, mask))
    for name, got, ref in zip(("O", "dQ", "dK", "dV"), (O, *grads), refs):
        check_tensor(name, to_f64(got), ref, bar_for(dtype))
