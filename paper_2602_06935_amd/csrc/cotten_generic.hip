// What the kernel families share on the host and around the states: the launch plan, the
// three-launch structure of the kernels for wide rows (partial states -> fixed-order reduction ->
// apply), the reduction kernel itself, <S, dS> for d loss / d log(scale), and the kernels of
// the learnable normaliser.
#include "cotten_launch.h"

namespace cotten {
namespace {

constexpr int kThreads = 256;

// Sums the partial states of every slice in split order (fixed order => results do
// not depend on scheduling).  One thread per four state elements; the loads of kAhead splits travel
// together.  Bound by the reads of the partials, out of the memory-side cache (one float per
// thread, one split at a time: forward of 8 slices x 3000 rows, 16-bit d = 128, 22.9 us against 20.6).  The splits of a
// batch are summed before they join the sum: with one chain over 63 splits its roundings were most of the error.
__global__ __launch_bounds__(kThreads) void reduce_states_kernel(
    const float4* __restrict__ partial, float4* __restrict__ reduced, int splits, int quads,
    size_t total) {
  constexpr int kAhead = 8;
  const size_t e = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (e >= total) return;
  const size_t bh = e / quads, k = e % quads;
  const float4* __restrict__ src = partial + bh * splits * quads + k;
  float4 s = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int p0 = 0; p0 < splits; p0 += kAhead) {
    float4 v[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      v[i] = p0 + i < splits ? src[static_cast<size_t>(p0 + i) * quads] : float4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 1; i < kAhead; ++i)
      if (p0 + i < splits) {
        v[0].x += v[i].x;
        v[0].y += v[i].y;
        v[0].z += v[i].z;
        v[0].w += v[i].w;
      }
    s.x += v[0].x;
    s.y += v[0].y;
    s.z += v[0].z;
    s.w += v[0].w;
  }
  reduced[e] = s;
}

// dlog[bh] = scale_bh * <S_bh, dS'_bh> with dS' = sum_i qhat_i^T dO_i (the states in the
// workspace carry no scale), i.e. <S, dS> = sum_i dO_i . O_i.  One workgroup per slice; the
// sum runs in a fixed order (strided per thread, then a tree over the threads).
__global__ __launch_bounds__(kThreads) void state_inner_product_kernel(
    const float* __restrict__ states, const float* __restrict__ dstates, int dd, float scale,
    const float* __restrict__ slice_scale, float* __restrict__ dlog) {
  __shared__ float part[kThreads];
  const size_t off = static_cast<size_t>(blockIdx.x) * dd;
  float s = 0.0f;
  for (int e = threadIdx.x; e < dd; e += kThreads) s += states[off + e] * dstates[off + e];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if (static_cast<int>(threadIdx.x) < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0)
    dlog[blockIdx.x] = part[0] * (slice_scale != nullptr ? slice_scale[blockIdx.x] : scale);
}

// slice_scale[b*H+h] = n_b^(-m_h) = exp2(-m_h log2 n_b)
__global__ __launch_bounds__(kThreads) void normaliser_fwd_kernel(
    const float* __restrict__ m, const int32_t* __restrict__ n, float* __restrict__ slice_scale,
    int B, int H, int N) {
  const int e = blockIdx.x * kThreads + threadIdx.x;
  if (e >= B * H) return;
  const float nb = static_cast<float>(n != nullptr ? n[e / H] : N);
  slice_scale[e] = exp2f(-m[e % H] * log2f(nb));
}

// dm[h] = -sum_b ln(n_b) dlog[b*H+h]: one workgroup per head, fixed order (strided per
// thread, then a tree over the threads).
__global__ __launch_bounds__(kThreads) void normaliser_bwd_kernel(
    const float* __restrict__ dlog, const int32_t* __restrict__ n, float* __restrict__ dm, int B,
    int H, int N) {
  __shared__ float part[kThreads];
  const int h = blockIdx.x;
  float s = 0.0f;
  for (int b = threadIdx.x; b < B; b += kThreads)
    s += logf(static_cast<float>(n != nullptr ? n[b] : N)) * dlog[static_cast<size_t>(b) * H + h];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if (static_cast<int>(threadIdx.x) < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) dm[h] = -part[0];
}

// Where the reduced states live: behind the partials when a reduction
// is needed, otherwise the single partial of each slice already is the state.
const float* reduce_generic(const Problem& p, const Plan& plan, int nstates) {
  if (plan.splits == 1) return p.workspace;
  const size_t BH = static_cast<size_t>(p.B) * p.H;
  const int dd = p.D * p.D;
  float* reduced = p.workspace + BH * plan.splits * dd * nstates;
  // S and dS partials are contiguous [nstates][BH*splits][dd]: one launch covers both
  launch_reduce_states(p.workspace, reduced, plan.splits, dd, BH * nstates, p.stream);
  return reduced;
}

// The three-launch structure of the matrix-core kernels for wide rows (cotten_wide.hip): partial
// states, their reduction, the kept state, the apply kernels, <S, dS>; one launch per direction
// where the sequence is not cut.
hipError_t run_wide(const Problem& p, const Plan& plan, bool bwd) {
  if (wide_fused_applies(p.dtype, p.B, p.H, plan.splits, bwd)) return launch_wide_fused(p, plan, bwd);
  const int BH = p.B * p.H;
  const int dd = p.D * p.D;
  if (hipError_t err = launch_wide_states(p, plan, bwd)) return err;
  const float* states = reduce_generic(p, plan, bwd ? 2 : 1);
  const size_t second = static_cast<size_t>(BH) * plan.splits * dd;
  const float* dstates =
      bwd ? states + (plan.splits == 1 ? second : static_cast<size_t>(BH) * dd) : nullptr;
  if (!bwd && p.saved_state != nullptr)
    launch_reduce_states(states, p.saved_state, 1, dd, static_cast<size_t>(BH), p.stream);
  if (hipError_t err = launch_wide_apply(p, plan, states, dstates, bwd)) return err;
  if (bwd && p.dlog_scale != nullptr)
    hipLaunchKernelGGL(state_inner_product_kernel, dim3(static_cast<unsigned>(BH)),
                       dim3(kThreads), 0, p.stream, states, dstates, dd, p.scale, p.slice_scale,
                       p.dlog_scale);
  return hipGetLastError();
}

}  // namespace

void launch_reduce_states(const float* partial, float* reduced, int splits, int dd, size_t slices,
                          hipStream_t stream) {
  // states are 16-byte aligned: so are the workspace and the caller's array (checked at the entry points),
  // and dd is a multiple of 1024 here (wide rows: D = 64 or 128)
  const int quads = dd / 4;
  const size_t total = slices * quads;
  const dim3 grid(static_cast<unsigned>((total + kThreads - 1) / kThreads), 1, 1);
  hipLaunchKernelGGL(reduce_states_kernel, grid, dim3(kThreads), 0, stream,
                     reinterpret_cast<const float4*>(partial), reinterpret_cast<float4*>(reduced), splits, quads,
                     total);
}

namespace {

// Workgroups per slice of a sequence that is cut (rows of up to 128 bytes).  The slices are dealt to the eight XCDs, and
// with them all their workgroups: what has to fit is `per_xcd` * splits on 32 compute units.  In 16 bits every workgroup
// of an apply launch gathers a partial state of 16 KB per split, as much as 128 rows of a tensor: that many splits and
// no more than about sqrt(N / 7) (or ten), and one workgroup per compute unit, two where a workgroup would have more than 600 rows
// or the slices are too many to fill one well.  Partial states of fp32 rows are a quarter of that: two workgroups per compute
// unit, or three where these fill it better.  Forward / backward, us, against as many splits as make 512 workgroups in all:
//   bf16 d = 64:  4 x 4096, 16 splits 13.8 / 26.8 (64: 29.4 / 56.3);  8 x 1500, 12: 11.7 / 21.4 (24: 12.5 / 22.5);  20 x 1500, 8: 13.2 /
//   24.6 (24: 23.5 / 45.9);  24 x 4096, 10: 18.7 / 40.0 (22: 28.3 / 57.3);  40 x 4096, 12: 25.5 / 49.6, 6: 24.0 / 51.6 (13: 30.8 / 65.3);
//   64 x 2000, 4: 19.8 / 40.9 (8: 20.9 / 43.3);  64 x 4096, 4: 37 / 67, 8: 34 / 71;  100 x 2500, 4: 34.7 / 65.5 (6: 37.1 / 80.7);
//   240 x 4096, 2: 108 / 241 (3: 117 / 267)
//   fp32 d = 32:  4 x 4096, 32: 11.1 / 19.9 (64: 12.9 / 23.4);  60 x 3333, 8: 24.6 / 53.6 (9: 26.7 / 57.2);  90 x 4096, 8: 49.2 / 98.4 (6:
//   53.6 / 107);  180 x 4096, 4: 85 / 188 (3: 94 / 213)
long split_count(long BH, long N, int dtype) {
  constexpr long kXcds = 8, kUnits = 32;  // and compute units of an XCD
  const long per_xcd = (BH + kXcds - 1) / kXcds, one = kUnits / per_xcd, two = 2 * kUnits / per_xcd, three = 3 * kUnits / per_xcd;
  long splits;
  if (dtype != 0) {
    splits = per_xcd > 8 || N > 600 * one ? two : one;
    long most = 10;
    while (7 * (most + 1) * (most + 1) <= N) ++most;
    if (splits > most) splits = most;
  } else if (per_xcd <= 2) {
    splits = one;
  } else {
    splits = 200 * three > 318 * two ? three : two;  // (fills 6 % more)
  }
  return splits < 2 ? 2 : splits;
}

constexpr long kUnits = 256;  // compute units

// Wide rows: parts of a sequence for fewer slices than compute units.  A part costs a d x d state (64 KB at d = 128) written,
// summed up and read back, and two launches more; whole sequences take one launch per direction (16-bit backward over
// fewer than 86 slices: three).  Forward / backward, us.

// bf16 d = 128.  Up to 128 slices: parts of 256 rows or more, one workgroup per compute unit, two for sequences of 4096 rows, and
// of 2048 where one leaves a fifth of the chip idle:
//   100 x 600 28 / 56 (3 parts, more workgroups than units: 34 / 61);  100 x 3000, 5: 81 / 204 (2: 86 / 216);  64 x 3000, 4: 53 / 137
//   (8: 60 / 143);  128 x 6000, 4: 167 / 467 (2: 172 / 458).
// Forward: whole for short sequences:
//   64 x 300 13.2 (2 parts 20.7);  64 x 600 20.8 (3: 22.3);  128 x 600 22.3 (2: 30.1);  85 x 800, 3: 28.4 (1: 29.7, 2: 28.8);  128 x 1300 61 (2: 53);
//   64 x 4096, 4 parts 70 (8: 78);  85 x 4096, 3: 88 (6: 95);  24 x 4096, 10: 34 (21: 40).
// More than 128 slices: whole, or from a length on three parts (140 x 4096 173 whole, 140 in three).
// Backward: the three roles of the last launch are workgroups of their own, so that as many parts as make 256 of them fill
// the chip; beyond a length (the shorter the less they fill it) 512, and beyond 700 rows each one part per compute unit:
//   64 x 300 21.5 whole (2: 28.2);  64 x 900 47.6 (4: 53.4);  85 x 1500 93 (3: 102);  48 x 600 32.0 (3: 33.8);  48 x 900, 3: 39.6 (1: 46.4,
//   4: 46.3);  24 x 900, 3: 26.7 (4: 30.4);  32 x 1500, 4: 41.4 (2: 43.6, 6: 46.2);  16 x 2500, 10: 35.6 (6: 42.6);  64 x 2500, 4: 125 (2: 138);
//   32 x 4096, 8: 108 (16: 117).
// From 86 slices on one launch, whole up to a length: 128 x 600 57 (2: 64);  128 x 1300 109 (2: 127);  110 x 1300 105 (2: 118);  90 x 600
// 56 (2: 52);  140 x 900 79 (3: 112);  200 x 1800 192 (whole in the kernel before: 257);  160 x 2500 241 (3: 265);  140 x 2500 242 (3: 241).
long wide_splits16(long BH, long N, bool bwd) {
  if (BH > 128) {
    if (bwd) return BH >= 140 || N <= 1900 ? 1 : 3;
    return N >= 50 * (BH - 100) ? 3 : 1;
  }
  const long one = kUnits / BH, two = 2 * kUnits / BH;
  const bool crowded = N >= 4096 || (N >= 2048 && 5 * one * BH < 4 * kUnits);
  const long long_parts = (N + 255) / 256, most = (crowded ? two : one) < long_parts ? (crowded ? two : one) : long_parts;
  if (!bwd) {
    if (N <= 6 * BH + 260) return 1;
    return BH >= 86 || N >= 5000 || one > most ? most : one;
  }
  if (BH >= 86) {
    const long whole = 55 * (BH - 85) < 1900 ? 55 * (BH - 85) : 1900;
    return N <= 400 || N <= whole ? 1 : most;
  }
  const long few = kUnits / (3 * BH), fill = 3 * BH * few;  // of 256
  long parts;
  if (N <= 256 * few || N <= 100 + 1800 * fill * fill / (kUnits * kUnits)) {
    parts = BH >= 20 && N <= 260 + 2 * BH ? 1 : few;
  } else {
    const long more = 2 * kUnits / (3 * BH);
    if (N > 700 * more) parts = N >= 5000 ? two : one;
    else parts = more < N / 200 ? more : N / 200;
  }
  return parts < most ? parts : most;
}

// fp32 rows, one workgroup of eight waves per compute unit (d = 128), or up to three of four (d = 64).
// d = 128:  forward 250 x 300 41.9 whole (2 parts 72);  200 x 1000 110 (2: 140);  128 x 1000, 2: 82 (4: 95);  64 x 1800, 4: 80 (8: 93);
//   4 x 1000, 16: 20.6 (4: 33);  1 x 16000, 63: 40 (42: 49);  backward 128 x 1000 168 whole (4: 227);  250 x 600 174 (2: 246);  90 x 1800 248
//   (6: 256);  64 x 1800, 2: 174 (7: 217);  4 x 6000, 19: 52 (32: 55);  8 x 6000, 16: 80 (10: 85);  16 x 4000, 8: 108 (5: 123, 16: 115);
//   32 x 4000, 4: 191 (5: 200);  32 x 6000, 8: 269 (4: 278).
//   More than half as many slices as compute units, beyond a length, and other counts that leave much of the chip idle (whole or in few parts):
//   forward 129 x 1700, 3: 145 (1: 167, 4: 153);  150 x 3000, 3: 242 (1: 285);  170 x 4096, 3: 334 (1: 384);  180 x 1700 171 (3: 186);
//   92 x 2500, 5: 137 (2: 160);  100 x 4096, 5: 208 (2: 223);  backward 129 x 950, 3: 195 (1: 228);  129 x 3000, 3: 498 (1: 709);  150 x 1150,
//   3: 249 (1: 266);  170 x 3000, 3: 625 (1: 733);  180 x 2040, 3: 469 (1: 500);  192 x 1700 424 (3: 428);  92 x 3000, 5: 365 (1: 392);
//   100 x 2040 267 (5: 285);  72 x 1700, 3: 183 (1: 218);  85 x 950 128 (3: 132);  85 x 1400, 3: 179 (1: 189);  46 x 330, 2: 47.6 (1: 51.3);
//   58 x 400 56.5 (2: 57.2);  46 x 1700, 5: 129 (2: 138);  58 x 2500, 4: 213 (2: 224);  64 x 1700, 2: 160 (4: 168);  36 x 3000, 7: 162 (3: 180).
// d = 64:  forward 250 x 600 38 whole (2: 45);  150 x 1800, 3: 74 (4: 81);  90 x 3500, 8: 81 (6: 90);  64 x 1800, 4: 36 (7: 37);  10 x 1000,
//   8: 13.7 (4: 17.4);  64 x 320 16.5 (3: 15.7);  80 x 320 16.7 (3: 17.1);  64 x 4000, 8: 68 (4: 73, 9: 73);  197 x 1916, 3: 95 (2: 106);  32 x 6000, 16: 53 (24: 54,
//   8: 56);  backward 128 x 1000 73 whole (4: 87);  250 x 600 86 (2: 109);  200 x 1800, 3: 211 (1: 220);  32 x 1000, 8: 27 (4: 29);
//   64 x 1800, 4: 73 (7: 82);  64 x 3500, 11: 143 (4: 147);  20 x 1000, 4: 21.2 (8: 22.4);  4 x 4000, 21: 21 (32: 23);  8 x 8000, 32: 42
//   (16: 49);  just over half as many slices as units, 129 x 680, 2: 59 (1: 65);  140 x 950, 2: 91 (1: 104);  150 x 800, 2: 73 (1: 79);  129 x 800, 2:
//   62.5 (1: 60.4);  140 x 560 53.7 (2: 54.2);  160 x 950 99 (2: 101).  Forward of 154 ... 226 slices, whole up to 1150 rows:  154 x 1034
//   41 (4: 45);  165 x 1100 51.1 (4: 52.1);  176 x 1034 48 (4: 58);  183 x 1034 45.7 (4: 57.7; errors 1.46e-7 and 1.48e-7);  192 x 1150 61.3 (4:
//   64.8), x 1200 65.6 (4: 60.6);  205 x 1150 63.8 (3: 64.9).  (The forward of 32 x 3600 is faster in 15 parts of 256 rows, 33 to 39, but
//   these are not summed apart: error 1.8e-7 against 1.5e-7.)
long wide_splits32(long BH, long N, int D, bool bwd) {
  if (N <= 256) return 1;  // (calls of this length need no workspace)
  // workgroups per slice: one per compute unit in all, two, three, and those of a launch of three roles
  const long one = kUnits / BH, two = 2 * kUnits / BH, three = 3 * kUnits / BH, few = BH >= 86 ? 1 : kUnits / (3 * BH);
  // 64 rows or more each, and 256 where the partial states would be more than 48
  const long long_parts = (N + 255) / 256, most = N <= 48 * 64 ? (N + 63) / 64 : long_parts < 48 ? 48 : long_parts;
  const auto up_to = [](long parts, long limit) { return parts < limit ? parts : limit; };
  if (D == 128) {
    if (!bwd) {
      if (BH > 128) return BH <= 170 && N > 1400 ? 3 : 1;
      return one == 2 && N <= 330 ? 1 : up_to(two == 5 && N > 2000 ? two : one, most);
    }
    if (BH > 128) return BH <= 192 && N > 700 + 12 * (BH - 129) ? 3 : 1;
    if (BH >= 86) return two == 5 && N > 125 * BH - 9100 ? two : 1;
    if (BH > 64) return N > 1000 ? one : 1;
    if (BH > 42) return N > 100 * BH - 3500 ? one : N > (BH <= 56 ? 300 : 450) ? 2 : 1;
    return up_to(N * BH > 180000 || (BH > 32 && N > 2400) ? one : N > 450 * few ? one / 2 : few, most);
  }
  if (!bwd) {
    long far = one == 1 ? 1300 * BH / kUnits : 550 * one;
    if (BH >= 154 && far < 1150) far = 1150;
    if (N > far) return up_to(one == 1 || 200 * three > 318 * two ? three : two, long_parts);
    return N <= 200 + 2 * BH ? 1 : up_to(one, most);
  }
  if (BH > 128 && BH <= 150 && N > 600 && N <= 8 * BH) return 2;
  if (N <= (BH > 128 ? 8 * BH : BH >= 86 ? 1100 + 60 * (BH - 86) : few == 1 ? 420 : 0)) return 1;
  if (BH >= 86 || N > 600 * (N > 250 * few ? one : few)) return up_to(three, long_parts);
  return up_to(N > 250 * few ? one : few, most);
}

// fp32 rows: calls that are cut for speed but run whole, in one launch, where there is no workspace.
bool whole_without_workspace32(long BH, long N, int D, bool bwd) {
  if (D < 128) return D == 64 && bwd && BH > 128 && N <= 8 * BH;
  if (!bwd) return BH > 128;
  return BH > 85 || (BH > 64 ? N * BH <= 180000 : BH > 42 && N <= 450);
}

}  // namespace

Plan make_plan(int B, int H, int N, int D, int dtype, bool is_bwd, size_t given) {
  const long BH = static_cast<long>(B) * H;
  const size_t nstates = is_bwd ? 2 : 1;
  Plan plan;
  constexpr long kBlock = 64, kMostRows = 2048;  // of a workgroup, up to 128 bytes each: their key flags
  const auto blocks_of = [&](long parts) {
    const long r = (N + parts - 1) / parts;
    return (r + kBlock - 1) / kBlock * kBlock;
  };
  const auto parts_of = [&](long r) { return (N + r - 1) / r; };
  long splits, rows;
  if (mfma_supports(dtype, D)) {
    // One workgroup per slice and launch while that fills enough of the chip or the slice is short; otherwise the
    // sequence is cut, in blocks of 64 rows (split_count).
    // 16-bit sequences that fit LDS go to the resident kernels - except the forward of the
    // longer ones when there are many slices, where the fused kernel that keeps its tiles in
    // registers is faster (N = 208, 512 slices: 9.6 against 10.2 us; the resident kernel wins
    // at N = 100, 7.1 against 7.6 us, and with 64 slices, 5.7 against 7.2 us).
    const bool fused_fwd_instead = !is_bwd && N > 160 && BH >= 256;
    if (resident_supports(dtype, D, N) && !fused_fwd_instead) {
      plan.path = Plan::kResident;
      plan.splits = 1;
      plan.rows_per_split = N;
      plan.workspace_floats = 0;
      return plan;
    }
    // Long sequences stay on one workgroup per slice as well when there are slices enough
    // (measured at N = 3000 ... 4096: the backward from 256 slices on, the forward from 512).
    constexpr long kFusedLongMaxN = 16384;  // key flags of the slice must fit LDS
    const bool fused_long = N <= kFusedLongMaxN && BH >= (is_bwd ? 256 : 512);
    // One launch against two or three, forward / backward, us, whole and cut: bf16 d = 64: 40 x 320 rows 9.8 / 18.6, 10.4 / 18.4;
    // 64 x 420 11.7 / 23.6, 11.5 / 21.4;  100 x 420 12.0 / 24.2, 14.5 / 26.8;  100 x 600 15.5 / 30.5, 15.4 / 30.9;  130 x 900 21.3 / 44.3,
    // 20.0 / 42.3;  160 x 900 22.6 / 45.3, 21.4 / 45.5;  160 x 1300 34 / 65, 26 / 55;  200 x 1300 35 / 65, 38 / 67;  200 x 2000 51 / 105,
    // 54 / 111.  fp32 d = 32: 100 x 260 10.4 / 19.3, 10.4 / 18.6;  130 x 320 10.8 / 20.3, 11.5 / 21.1;  160 x 420 13.8 / 26.0, 13.4 /
    // 26.4;  200 x 600 19.0 / 35.0, 18.6 / 36.1;  250 x 600 20.1 / 36.9, 20.5 / 41.7;  250 x 900 27.5 / 55.9, 26.5 / 55.0.
    // fp32, beyond 320 rows and up to 168 slices (three workgroups of each on two per compute unit):  128 x 330, 3 parts: 11.1 / 20.6, whole 11.7 /
    // 22.1;  160 x 470, 3: 13.5 / 25.6, whole 14.2 / 28.1;  170 x 470, 2: 14.1 / 28.6, whole 14.3 / 28.0.  (Whole also there, without a workspace for two.)
    const auto at_most = [](long x, long limit) { return x < limit ? x : limit; };
    const long enough = dtype != 0 ? at_most(N / 5 - 10, 170) : at_most(N / 4 + 40, 256);
    const bool three = dtype == 0 && N > 320 && BH <= 168 && given / 2 >= nstates * BH * mfma_state_dim(dtype) * mfma_state_dim(dtype);
    if ((N <= kMostRows && ((BH >= enough && !three) || N <= 256)) || fused_long) {
      plan.path = Plan::kFused;
      plan.splits = 1;
      plan.rows_per_split = N;
      plan.workspace_floats = 0;
      return plan;
    }
    plan.path = Plan::kSplit;
    splits = split_count(BH, N, dtype);
    const long by_len = (N + kMostRows - 1) / kMostRows;
    if (splits < by_len) splits = by_len;
    const long max_splits = (N + kBlock - 1) / kBlock;
    if (splits > max_splits) splits = max_splits;
    rows = blocks_of(splits);
  } else {
    // Wide rows (256 or 512 bytes), in blocks of 64 rows.
    plan.path = Plan::kGeneric;
    splits = BH >= kUnits ? 1 : dtype == 0 ? wide_splits32(BH, N, D, is_bwd) : wide_splits16(BH, N, is_bwd);
    if (splits < 1) splits = 1;
    rows = blocks_of(splits);
  }
  if (dtype == 0 && parts_of(rows) > 1) {  // a smaller workspace than is asked for: as many parts as it holds
    const bool wide = plan.path == Plan::kGeneric;
    const size_t side = wide ? D : mfma_state_dim(dtype), part = static_cast<size_t>(BH) * side * side * nstates;
    const long sum = wide ? 1 : 0;  // (wide rows: and their sum)
    const long held = given / part > static_cast<size_t>(N) ? N : static_cast<long>(given / part) - sum;
    const long least = wide || N <= 2 * kMostRows ? 2 : parts_of(kMostRows);
    if (parts_of(rows) > held) {
      if (held >= least) rows = blocks_of(held);
      else if (whole_without_workspace32(BH, N, D, is_bwd)) rows = blocks_of(1);
    }
  }
  splits = parts_of(rows);
  plan.splits = static_cast<int>(splits);
  plan.rows_per_split = static_cast<int>(rows);
  if (plan.path == Plan::kSplit) {
    const size_t side = mfma_state_dim(dtype);
    plan.workspace_floats = static_cast<size_t>(BH) * side * side * splits * nstates;
  } else {
    // partial states, plus the reduced states when there is more than one partial
    // (one launch per direction: the state never leaves the compute unit)
    plan.workspace_floats =
        wide_fused_applies(dtype, B, H, static_cast<int>(splits), is_bwd)
            ? 0
            : static_cast<size_t>(BH) * D * D * nstates * (splits + (splits > 1 ? 1 : 0));
  }
  return plan;
}

hipError_t launch_generic_fwd(const Problem& p, const Plan& plan) {
  return wide_supports(p.dtype, p.D) ? run_wide(p, plan, false) : hipErrorInvalidValue;
}

hipError_t launch_generic_bwd(const Problem& p, const Plan& plan) {
  return wide_supports(p.dtype, p.D) ? run_wide(p, plan, true) : hipErrorInvalidValue;
}

hipError_t launch_normaliser_fwd(const float* m, const int32_t* n, float* slice_scale, int B,
                                 int H, int N, hipStream_t stream) {
  const unsigned blocks = static_cast<unsigned>((static_cast<long>(B) * H + kThreads - 1) / kThreads);
  hipLaunchKernelGGL(normaliser_fwd_kernel, dim3(blocks), dim3(kThreads), 0, stream, m, n,
                     slice_scale, B, H, N);
  return hipGetLastError();
}

hipError_t launch_normaliser_bwd(const float* dlog, const int32_t* n, float* dm, int B, int H,
                                 int N, hipStream_t stream) {
  hipLaunchKernelGGL(normaliser_bwd_kernel, dim3(static_cast<unsigned>(H)), dim3(kThreads), 0,
                     stream, dlog, n, dm, B, H, N);
  return hipGetLastError();
}

}  // namespace cotten
