// Matrix-core kernels for 256-byte rows of 16-bit elements: bf16 / fp16 I/O with d_h = 128 (d_model = 256
// with two heads, "Sequence Length and Embedding Size").  (fp32 rows of 256 and 512 bytes:
// cotten_wide32.hip; the entry points at the end of this file hand over to it.)
//
// A 256-byte row is handled as two 128-byte halves, a d_h x d_h state as four quadrants of
// the size the 128-byte-row formats work on (cotten_mfma_core.h), so that their tile layout,
// MFMA products, operand images and row epilogues serve unchanged:
//
//     S[p][q] = sum_j khat_j[half p]^T v_j[half q]           (state kernel)
//     O[half q] = sum_p Qhat[half p] S[p][q]                 (apply kernels; likewise dQ, dK, dV)
//
// with the row norm taken over both halves.  Three launches (partial states in the caller's
// workspace, [kinds][slices * splits][D * D] floats, then the reduced states):
//
//   wide_state_kernel   a workgroup of four (or eight) waves reduces its share of the rows of a slice
//                       to a partial state: per round every wave stages one 16-row tile in LDS,
//                       then wave (p, q) adds four tiles of the round to its quadrant (with eight
//                       waves two waves share a quadrant and their sums meet at the end)
//   (the partial states of a slice are summed in split order by reduce_states_kernel)
//   wide_fwd_kernel / wide_bwd_kernel
//                       a workgroup builds the operand images of the state it needs from the
//                       reduced state, then every wave streams 16-row tiles through a private
//                       LDS tile set: products per quadrant, epilogue per half row, 128-bit
//                       stores.  The backward runs dQ, dV and dK as three roles of one launch
//                       (blockIdx.y), each with the one set of images it needs.
#include "cotten_launch.h"
#include "cotten_mfma_core.h"

namespace cotten {
namespace {
namespace wide {

using namespace mfma;

// Every kernel exists for workgroups of 4 and of 8 waves (template parameter WAVES): 4 when there
// are workgroups enough to put two on every compute unit, 8 when there are not.
//
constexpr int P = 2;                     // 128-byte pieces of a row
constexpr int kHalfBytes = kRowBytes;    // one piece of a row

// A 16-row tile of a tensor pair in the load layout: piece [h][c] is bytes 128 c + 16 ch .. + 15 of
// row r8 + 8 h.  `live` bit h: the row takes part.
struct WideRaw {
  u32x4_t x[2][P], y[2][P];
  int live;
};

// The two tensors of a pass as buffer resources over one slice (see Src in cotten_mfma_core.h:
// lanes whose row does not take part get zeros and cause no traffic).
struct WideSrc {
  __amdgpu_buffer_rsrc_t x, y;
  int stride;
  __device__ __forceinline__ WideSrc(const unsigned char* X, const unsigned char* Y, int N, int stride_bytes)
      : stride(stride_bytes) {
    const int bytes = N > 0 ? (N - 1) * stride + P * kHalfBytes : 0;
    x = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(X), 0, bytes, 0x00020000);
    y = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(Y), 0, bytes, 0x00020000);
  }
};

// Bit h: row row0 + r8 + 8 h is below `limit` and, if a mask is given, a valid key.
__device__ __forceinline__ int row_bits(const uint8_t* __restrict__ mask, int row0, int limit,
                                        const Lane& L) {
  int bits = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = row0 + L.r8 + 8 * h;
    if (row < limit) bits |= static_cast<int>(mask == nullptr || mask[row] != 0) << h;
  }
  return bits;
}

template <bool USE_Y>
__device__ __forceinline__ void load_wide(WideRaw& r, const Lane& L, const WideSrc& src, int row0,
                                          int bits) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const bool live = ((bits >> h) & 1) != 0;
    const uint32_t off =
        live ? static_cast<uint32_t>(row0 + L.r8 + 8 * h) * src.stride + L.ch * 16 : kOutOfBuffer;
#pragma unroll
    for (int c = 0; c < P; ++c) {
      r.x[h][c] = __builtin_amdgcn_raw_buffer_load_b128(src.x, off + c * kHalfBytes, 0, 0);
      if (USE_Y) r.y[h][c] = __builtin_amdgcn_raw_buffer_load_b128(src.y, off + c * kHalfBytes, 0, 0);
      else r.y[h][c] = u32x4_t{0, 0, 0, 0};
    }
  }
  r.live = bits;
}

// The tile into LDS as 2 P tiles of 16 x 128 bytes [x pieces | y pieces] (each in the layout of
// cotten_mfma_core.h); x raw, normalised over the whole row, or through the element-wise map of
// the format (XMODE, see stage() in cotten_mfma_core.h).
// inv[h] = 1/r of row r8 + 8 h (0, with MARK -0, for a row that does not take part; with the element-wise map 1
// for a row that does, and a row that does not is written as zeros explicitly: phi(0) is not 0).
template <class F, int XMODE, bool USE_Y, bool MARK = false>
__device__ __forceinline__ void stage_wide(const WideRaw& r, const Lane& L, float eps,
                                           unsigned char* tiles, float (&inv)[2]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float f[P][F::EPL];
    const bool live = ((r.live >> h) & 1) != 0;
    const int off = (L.r8 + 8 * h) * kTileStride + L.ch * 16;
    if (XMODE == kXFeature) {
      inv[h] = live ? 1.0f : MARK ? -0.0f : 0.0f;
#pragma unroll
      for (int c = 0; c < P; ++c) {
        F::unpack(r.x[h][c], f[c]);
#pragma unroll
        for (int i = 0; i < F::EPL; ++i) f[c][i] = elu1_or_zero(f[c][i], live);
        *reinterpret_cast<u32x4_t*>(tiles + c * kTileBytes + off) = F::pack(f[c]);
        if (USE_Y) *reinterpret_cast<u32x4_t*>(tiles + (P + c) * kTileBytes + off) = r.y[h][c];
      }
      continue;
    }
    float ss = 0.0f;
#pragma unroll
    for (int c = 0; c < P; ++c) {
      F::unpack(r.x[h][c], f[c]);
#pragma unroll
      for (int i = 0; i < F::EPL; ++i) ss += f[c][i] * f[c][i];
    }
    inv[h] = inv_norm_or_zero<MARK>(row_sum8(ss), eps, live);
#pragma unroll
    for (int c = 0; c < P; ++c) {
      if (XMODE == kXNormalized) {
#pragma unroll
        for (int i = 0; i < F::EPL; ++i) f[c][i] *= inv[h];
        *reinterpret_cast<u32x4_t*>(tiles + c * kTileBytes + off) = F::pack(f[c]);
      } else {
        *reinterpret_cast<u32x4_t*>(tiles + c * kTileBytes + off) = r.x[h][c];
      }
      if (USE_Y) *reinterpret_cast<u32x4_t*>(tiles + (P + c) * kTileBytes + off) = r.y[h][c];
    }
  }
}

// How the x rows enter a product whose result is divided by r afterwards: raw under the cosine
// map (1/r applied to the result), mapped under the element-wise one (1/r is then 1).
template <class F>
constexpr int plain_mode() {
  return F::kMap == kMapElu1 ? kXFeature : kXRaw;
}

// 1/r of the tile's rows from the load layout to the product layout, through 16 floats of LDS.
__device__ __forceinline__ float inv_by_row(float* slot, const Lane& L, const float (&inv)[2]) {
  if (L.ch == 0) {
    slot[L.r8] = inv[0];
    slot[L.r8 + 8] = inv[1];
  }
  wave_lds_fence();
  return slot[L.i16];
}

// No row of the tile takes part (all of them masked or beyond the sequence): the wave can write
// the zeros such rows come out as without computing them.
__device__ __forceinline__ bool tile_dead(const WideRaw& r) {
  return __builtin_amdgcn_ballot_w64(r.live != 0) == 0;
}

template <class F>
__device__ __forceinline__ void store_zero_rows(unsigned char* out, int row0, int r_end, int stride,
                                                const Lane& L) {
  float z[2 * F::EPL];
#pragma unroll
  for (int i = 0; i < 2 * F::EPL; ++i) z[i] = 0.0f;
  const int row = row0 + L.i16;
  if (row < r_end) {
#pragma unroll
    for (int q = 0; q < P; ++q)
      store_product_row<F, kStoreStreamed>(out + q * kHalfBytes, row, RowAddr{stride, kHalfBytes}, L, z);
  }
}

extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

// ---- state kernel -------------------------------------------------------------------------------

// grid (slices * splits, 1 or 2): blockIdx.y == 1 reduces (Q, dO) to sum_i qhat_i^T dO_i instead
// of (K, V) under the key mask.  Partial states: row-major D x D floats per workgroup, the second
// kind `second_offset` floats behind the first.
// Each of the waves 0-3 of a group has one of the four blocks of the state (block i = piece i / P of x
// against piece i % P of y); with 8 waves two groups share the tiles of a round and their sums
// meet at the end.
template <class F, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void wide_state_kernel(
    const unsigned char* __restrict__ Q, const unsigned char* __restrict__ K,
    const unsigned char* __restrict__ V, const unsigned char* __restrict__ dO,
    const uint8_t* __restrict__ mask, float* __restrict__ ws, int H, int N, int splits,
    int rows_per_split, size_t second_offset, float eps, Strides st) {
  constexpr int Dh = F::D, D = P * Dh, kRoundRows = WAVES * TR;
  constexpr int kSetBytes = 2 * P * kTileBytes;  // the tiles one wave stages per round
  static_assert(WAVES == 4 || WAVES == 8, "one or two groups of four waves");
  unsigned char* round = smem;  // WAVES x [x pieces | y pieces]
  const Lane L;
  const int split = blockIdx.x % splits, bh = blockIdx.x / splits;
  const bool second = blockIdx.y == 1;
  const size_t base = st.slice_base(bh, H);
  const WideSrc src((second ? Q : K) + base, (second ? dO : V) + base, N, st.row.stride);
  const uint8_t* __restrict__ m =
      (second || mask == nullptr) ? nullptr : mask + static_cast<size_t>(bh / H) * N;
  // Forward (rows_per_split = 0): rounds are dealt to the workgroups in turn, so that padding at one end of the sequence is shared
  // evenly; backward: consecutive rows.  us, consecutive and dealt, bf16, lengths uniform in N/4 ... N, buffers in turn:  padded on the left, as
  // histories are, 16 slices x 3000 rows 25.3, 25.2;  32 x 3000 36.9, 35.5;  32 x 4096 44.4, 42.5;  64 x 4096 69.4, 67.0;  128 x 4096 122, 119;  on the right
  // 32 x 3000 37.3, 37.0;  32 x 4096 44.3, 45.4;  24 x 4096 38.2, 40.3 (the worst of 100 shapes);  128 x 4096 123, 123;  not padded +-1 %;  backward
  // 32 x 3000 79.2, 78.2 (no mask 71.4, 74.0); 8 x 1000 21.0, 21.5.  (Two rounds on their way, 32 x 3000: 3 % slower.)
  const bool dealt = rows_per_split == 0;
  const int step = dealt ? splits * kRoundRows : kRoundRows, begin = split * (dealt ? kRoundRows : rows_per_split);
  const int end = dealt || N < begin + rows_per_split ? N : begin + rows_per_split;
  // this wave's block of the state, and (8 waves) which four tiles of a round it adds up
  const int quadrant = L.wave & 3, part = L.wave >> 2;
  unsigned char* mine = round + L.wave * kSetBytes;

  typename F::Acc acc;
  acc.zero();
  const int first = begin + L.wave * TR;
  WideRaw cur;
  load_wide<true>(cur, L, src, first, row_bits(m, first, end, L));
  int next_bits = row_bits(m, first + step, end, L);
  for (int r0 = begin; r0 < end; r0 += step) {
    float inv[2];
    stage_wide<F, mapped_mode<F>(), true>(cur, L, eps, mine, inv);
    // the wave's tile of the next round travels while this round is added up
    load_wide<true>(cur, L, src, r0 + step + L.wave * TR, next_bits);
    next_bits = row_bits(m, r0 + 2 * step + L.wave * TR, end, L);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const unsigned char* tile = round + (4 * part + t) * kSetBytes;
      acc.mfma(tile + (quadrant / P) * kTileBytes, tile + (P + quadrant % P) * kTileBytes, L);
    }
    __syncthreads();  // the round's tiles are overwritten next
  }
  // 8 waves: the two sums of a block meet in LDS (the round buffer is free), in a fixed order
  f32x4_t* meet = reinterpret_cast<f32x4_t*>(round) + quadrant * F::Acc::kGroups * 64 + L.lane;
  static_assert(4 * F::Acc::kGroups * 64 * 16 <= 8 * kSetBytes, "the sums fit the round buffer");
  if (WAVES == 8) {
    if (part == 1) {
#pragma unroll
      for (int g = 0; g < F::Acc::kGroups; ++g) meet[g * 64] = acc.group(g);
    }
    __syncthreads();
    if (part == 1) return;
  }
  float* __restrict__ out =
      ws + (second ? second_offset : 0) + static_cast<size_t>(blockIdx.x) * D * D;
#pragma unroll
  for (int g = 0; g < F::Acc::kGroups; ++g) {
    f32x4_t v = acc.group(g);
    if (WAVES == 8) v += meet[g * 64];
    const int row = (quadrant / P) * Dh + F::Acc::group_row(g, L);
    const int col = (quadrant % P) * Dh + F::Acc::group_col(g, L);
#pragma unroll
    for (int i = 0; i < 4; ++i) out[(row + i) * D + col] = v[i];
  }
}

// ---- operand images --------------------------------------------------------------------------------

// The P x P block images of scale * M (M: a reduced state in global memory, row-major D x D),
// image (p, q) at images + (P p + q) * F::kImageBytes:
//   natural     op[m][n] = M[p Dh + m][q Dh + n]     for products that contract over n
//   transposed  op[n][m] = M[p Dh + m][q Dh + n]     for products that contract over m
template <class F, int WAVES, bool TRANSPOSED>
__device__ __forceinline__ void build_images(const float* __restrict__ M, float scale,
                                             unsigned char* images) {
  constexpr int Dh = F::D, D = P * Dh, kThreads = 64 * WAVES;
  // element pairs; the loads of a batch travel together
  constexpr int kPairs = D * D / 2, kBatch = kPairs / kThreads < 8 ? kPairs / kThreads : 8;
  static_assert(kBatch >= 1 && kPairs % (kBatch * kThreads) == 0, "state size");
  for (int e0 = threadIdx.x; e0 < kPairs; e0 += kBatch * kThreads) {
    float v0[kBatch], v1[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int e = e0 + j * kThreads;
      if (TRANSPOSED) {  // the pair (m, m + 1) of column n: consecutive threads take consecutive n
        const int m = 2 * (e / D), n = e % D;
        v0[j] = M[m * D + n];
        v1[j] = M[(m + 1) * D + n];
      } else {           // the pair (n, n + 1) of row m
        const int m = e / (D / 2), n = 2 * (e % (D / 2));
        const float2 v = *reinterpret_cast<const float2*>(M + m * D + n);
        v0[j] = v.x;
        v1[j] = v.y;
      }
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int e = e0 + j * kThreads;
      const int m = TRANSPOSED ? 2 * (e / D) : e / (D / 2);
      const int n = TRANSPOSED ? e % D : 2 * (e % (D / 2));
      unsigned char* image = images + (P * (m / Dh) + n / Dh) * F::kImageBytes;
      if (TRANSPOSED) F::write_image_pair(image, n % Dh, m % Dh, v0[j] * scale, v1[j] * scale);
      else F::write_image_pair(image, m % Dh, n % Dh, v0[j] * scale, v1[j] * scale);
    }
  }
}

// The P x P block operands of a role: held in registers for all the tiles of the wave (HOLD:
// 4 x 32 registers for the 16-bit formats with P = 2), or fetched from the images for every
// product (the backward roles share one kernel and do better at two waves per SIMD than with
// the operands held at one).
template <class F, bool HOLD>
struct Quadrants {
  typename F::Operand held[HOLD ? P * P : 1];
  const unsigned char* images;
  __device__ __forceinline__ Quadrants(const unsigned char* img, const Lane& L) : images(img) {
    if (HOLD) {
#pragma unroll
      for (int i = 0; i < P * P; ++i) held[i].load(images + i * F::kImageBytes, L);
    }
  }
  // out = sum_c X[piece c] W(first + c * step), images numbered P p + q
  __device__ __forceinline__ void apply(const typename F::TileRows (&X)[P], int first, int step,
                                        const Lane& L, float (&out)[2 * F::EPL]) const {
    f32x4_t a[F::NT];
#pragma unroll
    for (int c = 0; c < P; ++c) {
      if (HOLD) {
        if (c == 0) F::apply(X[c], held[first], a);
        else F::apply_onto(X[c], held[first + c * step], a);
      } else {
        typename F::Operand W;
        W.load(images + (first + c * step) * F::kImageBytes, L);
        if (c == 0) F::apply(X[c], W, a);
        else F::apply_onto(X[c], W, a);
      }
    }
    product_rows<F>(a, out);
  }
};

// ---- apply roles ------------------------------------------------------------------------------------

struct ApplyArgs {
  const unsigned char* X;   // Q or K
  const unsigned char* Y;   // dO or V (projected role), unused otherwise
  const uint8_t* mask;      // key mask of the slice's batch row, or nullptr
  const float* state;       // reduced state of the slice, row-major D x D
  unsigned char* out;       // O, dQ, dK or dV
  int N, r_begin, r_end, stride;
  float scale, eps;
};

// LDS of the apply kernels: [P x P images][per wave: 2 P tiles, 16 floats]
template <class F, int WAVES>
struct ApplyLds {
  static constexpr int kImages = 0;
  static constexpr int kWave = P * P * F::kImageBytes;
  static constexpr int kWaveBytes = 2 * P * kTileBytes + TR * 4;
  static constexpr int kBytes = kWave + WAVES * kWaveBytes;
};

// out rows = (x rows) M / r, contraction over the rows of M:  O = scale qhat S,  dV = scale khat dS.
// One tile of the plain role: `cur` staged raw into the wave's tile set, out rows = x W / r.
template <class F, bool HOLD>
__device__ __forceinline__ void plain_tile(const Quadrants<F, HOLD>& W, const WideRaw& cur, int row0,
                                           int r_end, unsigned char* out, int stride, float eps,
                                           unsigned char* tiles, const Lane& L) {
  if (tile_dead(cur)) {
    store_zero_rows<F>(out, row0, r_end, stride, L);
    return;
  }
  float* inv_slot = reinterpret_cast<float*>(tiles + 2 * P * kTileBytes);
  float inv[2];
  stage_wide<F, plain_mode<F>(), false>(cur, L, eps, tiles, inv);
  const float inv_r = inv_by_row(inv_slot, L, inv);
  typename F::TileRows X[P];
#pragma unroll
  for (int c = 0; c < P; ++c) X[c].load(tiles + c * kTileBytes, L);
  const int row = row0 + L.i16;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    float o[2 * F::EPL];
    W.apply(X, q, P, L, o);
#pragma unroll
    for (int i = 0; i < 2 * F::EPL; ++i) o[i] *= inv_r;
    if (row < r_end)
      store_product_row<F, kStoreStreamed>(out + q * kHalfBytes, row, RowAddr{stride, kHalfBytes}, L, o);
  }
  wave_lds_fence();
}

// `images`: the transposed block images of scale * M; `tiles`: this wave's tile set.
// The wave's first tile: requested here, or (REQUESTED) by the caller with request_first_tile.
template <int WAVES>
__device__ __forceinline__ void request_first_tile(WideRaw& cur, const ApplyArgs& a, const Lane& L) {
  const WideSrc src(a.X, a.X, a.N, a.stride);
  const int row0 = a.r_begin + L.wave * TR;
  load_wide<false>(cur, L, src, row0, row_bits(a.mask, row0, a.r_end, L));
}

template <class F, int WAVES, bool HOLD, bool REQUESTED = false>
__device__ __forceinline__ void plain_tiles(const ApplyArgs& a, const unsigned char* images,
                                            unsigned char* tiles, const Lane& L,
                                            const WideRaw* first = nullptr) {
  constexpr int kRoundRows = WAVES * TR;  // rows between two tiles of a wave
  const Quadrants<F, HOLD> W(images, L);
  const WideSrc src(a.X, a.X, a.N, a.stride);
  int row0 = a.r_begin + L.wave * TR;
  WideRaw cur;
  if (REQUESTED) cur = *first;
  else request_first_tile<WAVES>(cur, a, L);
  int next_bits = row_bits(a.mask, row0 + kRoundRows, a.r_end, L);
  for (; row0 < a.r_end; row0 += kRoundRows) {
    const WideRaw tile = cur;
    load_wide<false>(cur, L, src, row0 + kRoundRows, next_bits);
    next_bits = row_bits(a.mask, row0 + 2 * kRoundRows, a.r_end, L);
    plain_tile<F, HOLD>(W, tile, row0, a.r_end, a.out, a.stride, a.eps, tiles, L);
  }
}

template <class F, int WAVES, bool HOLD>
__device__ __forceinline__ void plain_role(const ApplyArgs& a) {
  const Lane L;
  unsigned char* images = smem + ApplyLds<F, WAVES>::kImages;
  unsigned char* tiles = smem + ApplyLds<F, WAVES>::kWave + L.wave * ApplyLds<F, WAVES>::kWaveBytes;
  build_images<F, WAVES, true>(a.state, a.scale, images);
  __syncthreads();
  plain_tiles<F, WAVES, HOLD, false>(a, images, tiles, L);
}

// The row epilogue of dQ and dK over all pieces of a row, E holding the mapped rows (xhat, or
// phi(x)):  cosine map  g <- (g - xhat (xhat . g)) / r;   ELU + 1  g <- g * phi'(x), phi' = min(phi, 1).
template <class F>
__device__ __forceinline__ void finish_projected(float (&g)[P][2 * F::EPL], typename F::TileRows (&E)[P],
                                                 float inv_r, const Lane& L) {
  if (F::kMap == kMapElu1) {
#pragma unroll
    for (int p = 0; p < P; ++p) feature_grad_rows<F>(g[p], E[p]);
    return;
  }
  float proj = 0.0f;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    float u[2 * F::EPL];
    E[p].unpack(u);
#pragma unroll
    for (int c = 0; c < 2 * F::EPL; ++c) proj += u[c] * g[p][c];
    E[p].forget_unpacked();
  }
  proj = row_sum_groups(proj, L);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    float u[2 * F::EPL];
    E[p].unpack(u);
#pragma unroll
    for (int c = 0; c < 2 * F::EPL; ++c) g[p][c] = (g[p][c] - u[c] * proj) * inv_r;
  }
}

// out rows = (g - xhat (xhat . g)) / r with g = (y rows) M^T, contraction over the columns of M:
//   dQ from (Q, dO) and scale S;   dK from (K, V) and scale dS (masked rows come out as zeros).
// `images`: the natural block images of scale * M.
template <class F, int WAVES>
__device__ __forceinline__ void projected_tiles(const ApplyArgs& a, const unsigned char* images,
                                                unsigned char* tiles, const Lane& L) {
  constexpr int kRoundRows = WAVES * TR;
  float* inv_slot = reinterpret_cast<float*>(tiles + 2 * P * kTileBytes);
  const Quadrants<F, false> W(images, L);
  const WideSrc src(a.X, a.Y, a.N, a.stride);
  int row0 = a.r_begin + L.wave * TR;
  WideRaw cur;
  load_wide<true>(cur, L, src, row0, row_bits(a.mask, row0, a.r_end, L));
  int next_bits = row_bits(a.mask, row0 + kRoundRows, a.r_end, L);
  for (; row0 < a.r_end; row0 += kRoundRows) {
    if (tile_dead(cur)) {  // nothing was fetched: zeros
      load_wide<true>(cur, L, src, row0 + kRoundRows, next_bits);
      next_bits = row_bits(a.mask, row0 + 2 * kRoundRows, a.r_end, L);
      store_zero_rows<F>(a.out, row0, a.r_end, a.stride, L);
      continue;
    }
    float inv[2];
    stage_wide<F, mapped_mode<F>(), true>(cur, L, a.eps, tiles, inv);
    load_wide<true>(cur, L, src, row0 + kRoundRows, next_bits);
    next_bits = row_bits(a.mask, row0 + 2 * kRoundRows, a.r_end, L);
    const float inv_r = inv_by_row(inv_slot, L, inv);
    typename F::TileRows Y[P], E[P];
#pragma unroll
    for (int c = 0; c < P; ++c) Y[c].load(tiles + (P + c) * kTileBytes, L);
    float g[P][2 * F::EPL];
#pragma unroll
    for (int p = 0; p < P; ++p)
      W.apply(Y, P * p, 1, L, g[p]);
#pragma unroll
    for (int c = 0; c < P; ++c) E[c].load(tiles + c * kTileBytes, L);
    finish_projected<F>(g, E, inv_r, L);
    const int row = row0 + L.i16;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      if (row < a.r_end)
        store_product_row<F, kStoreStreamed>(a.out + p * kHalfBytes, row, RowAddr{a.stride, kHalfBytes}, L, g[p]);
    }
    wave_lds_fence();
  }
}

template <class F, int WAVES>
__device__ __forceinline__ void projected_role(const ApplyArgs& a) {
  const Lane L;
  unsigned char* images = smem + ApplyLds<F, WAVES>::kImages;
  unsigned char* tiles = smem + ApplyLds<F, WAVES>::kWave + L.wave * ApplyLds<F, WAVES>::kWaveBytes;
  build_images<F, WAVES, false>(a.state, a.scale, images);
  __syncthreads();
  projected_tiles<F, WAVES>(a, images, tiles, L);
}

struct LaunchArgs {
  const unsigned char* Q;
  const unsigned char* K;
  const unsigned char* V;
  const unsigned char* dO;
  const uint8_t* mask;
  const float* states;   // reduced S of every slice
  const float* dstates;  // reduced sum_i qhat_i^T dO_i of every slice (backward)
  unsigned char* O;
  unsigned char* dQ;
  unsigned char* dK;
  unsigned char* dV;
  int H, N, splits, rows_per_split;
  float scale, eps;
  const float* slice_scale;
  Strides st;
};

__device__ __forceinline__ ApplyArgs role_args(const LaunchArgs& a) {
  ApplyArgs r{};
  const int split = blockIdx.x % a.splits, bh = blockIdx.x / a.splits;
  r.N = a.N;
  r.r_begin = split * a.rows_per_split;
  r.r_end = a.N < r.r_begin + a.rows_per_split ? a.N : r.r_begin + a.rows_per_split;
  r.stride = a.st.row.stride;
  r.scale = a.slice_scale != nullptr ? a.slice_scale[bh] : a.scale;
  r.eps = a.eps;
  return r;
}

template <class F, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void wide_fwd_kernel(const LaunchArgs a) {
  constexpr int D = P * F::D;
  const int bh = blockIdx.x / a.splits;
  const size_t base = a.st.slice_base(bh, a.H);
  ApplyArgs r = role_args(a);
  r.X = a.Q + base;
  r.mask = nullptr;  // queries are not masked
  r.state = a.states + static_cast<size_t>(bh) * D * D;
  r.out = a.O + base;
  plain_role<F, WAVES, true>(r);  // operands held in registers
}

// blockIdx.y: 0 dQ, 1 dV, 2 dK
template <class F, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void wide_bwd_kernel(const LaunchArgs a) {
  constexpr int D = P * F::D;
  const int bh = blockIdx.x / a.splits;
  const size_t base = a.st.slice_base(bh, a.H);
  ApplyArgs r = role_args(a);
  const uint8_t* keys = a.mask == nullptr ? nullptr : a.mask + static_cast<size_t>(bh / a.H) * a.N;
  if (blockIdx.y == 0) {
    r.X = a.Q + base;
    r.Y = a.dO + base;
    r.mask = nullptr;
    r.state = a.states + static_cast<size_t>(bh) * D * D;
    r.out = a.dQ + base;
    projected_role<F, WAVES>(r);
  } else if (blockIdx.y == 1) {
    r.X = a.K + base;
    r.mask = keys;
    r.state = a.dstates + static_cast<size_t>(bh) * D * D;
    r.out = a.dV + base;
    plain_role<F, WAVES, false>(r);
  } else {
    r.X = a.K + base;
    r.Y = a.V + base;
    r.mask = keys;
    r.state = a.dstates + static_cast<size_t>(bh) * D * D;
    r.out = a.dK + base;
    projected_role<F, WAVES>(r);
  }
}

// ---- one launch per direction: a workgroup of eight waves per slice ------------------------------
//
// When a sequence is not cut (one partial state per slice), the state need not leave the compute
// unit: the quadrant sums go from the accumulators straight into the operand images in LDS and
// the same workgroup streams the slice a second time through the apply roles.
//
//   forward   all eight waves reduce (K, V) to S (two waves per quadrant, rounds of 128 rows, the
//             sums meet in LDS), then stream Q through the transposed images of scale S.
//   backward  waves 0-3 reduce (K, V) to S, waves 4-7 (Q, dO) to dS, rounds of 64 rows each; then
//             all waves run dQ (natural images of S) and dV (transposed images of dS), and, the
//             images of S overwritten by the natural images of dS, dK.
//
// LDS: [SETS x four images][per wave: four tiles, 16 floats]; the tile sets double as the round
// buffer of the state phase and as the place where accumulators meet.
template <class F, int SETS, int WAVES = 8>
struct FusedLds {
  static constexpr int kWaves = WAVES;
  static constexpr int kSetBytes = 4 * F::kImageBytes;
  static constexpr int kTiles = SETS * kSetBytes;
  static constexpr int kWaveBytes = 4 * kTileBytes + TR * 4;
  static constexpr int kBytes = kTiles + kWaves * kWaveBytes;
  static_assert(WAVES == 4 || 4 * F::Acc::kGroups * 64 * 16 + 64 <= kWaves * kWaveBytes,
                "accumulators meet in the tile sets (four waves: each has a quadrant to itself)");
};

// The state phase of a group of four waves (wave & 3: the quadrant): every wave stages the 16 rows
// from `first_row` on of each round into its own tile set and adds the four tile sets of its group
// (wave >> 2) to its quadrant - or, `swapped`, the transposed sum (y tile)^T (x tile) with the two
// operands changing places, from which the natural image is the one that can be written
// straight from the lane.  Rows at and beyond N, and masked rows, are never fetched.
template <class F, int WAVE_BYTES>
__device__ __forceinline__ void fused_state_pass(typename F::Acc& acc, const WideSrc& src,
                                                 const uint8_t* __restrict__ m, int N, int first_row,
                                                 int round_rows, float eps, unsigned char* sets,
                                                 const Lane& L, bool swapped = false, int limit = -1) {
  if (limit < 0) limit = N;  // rows that exist (0: the group has no slice and only keeps step)
  const int quadrant = L.wave & 3, p = quadrant >> 1, q = quadrant & 1, group = L.wave >> 2;
  const int left = (swapped ? 2 + q : p) * kTileBytes, right = (swapped ? p : 2 + q) * kTileBytes;
  unsigned char* mine = sets + L.wave * WAVE_BYTES;
  acc.zero();
  WideRaw cur;
  load_wide<true>(cur, L, src, first_row, row_bits(m, first_row, limit, L));
  int next_bits = row_bits(m, first_row + round_rows, limit, L);
  for (int r0 = 0; r0 < N; r0 += round_rows) {
    float inv[2];
    stage_wide<F, mapped_mode<F>(), true>(cur, L, eps, mine, inv);
    load_wide<true>(cur, L, src, r0 + round_rows + first_row, next_bits);
    next_bits = row_bits(m, r0 + 2 * round_rows + first_row, limit, L);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const unsigned char* tile = sets + (4 * group + t) * WAVE_BYTES;
      acc.mfma(tile + left, tile + right, L);
    }
    __syncthreads();  // the tile sets are overwritten next
  }
}

// End of the forward's state phase: the two sums of a quadrant meet in `meet_area` (free by then),
// in a fixed order; the waves of the first group write the transposed images of scale * S and, if
// asked, S itself (row-major, for the caller's backward call).  Ends with a barrier.
template <class F>
__device__ __forceinline__ void forward_images(const typename F::Acc& acc, float scale,
                                               unsigned char* images, unsigned char* meet_area,
                                               float* __restrict__ kept, const Lane& L) {
  constexpr int Dh = F::D, D = 2 * Dh;
  const int quadrant = L.wave & 3, part = L.wave >> 2;
  f32x4_t* meet = reinterpret_cast<f32x4_t*>(meet_area) + quadrant * F::Acc::kGroups * 64 + L.lane;
  if (part == 1) {
#pragma unroll
    for (int g = 0; g < F::Acc::kGroups; ++g) meet[g * 64] = acc.group(g);
  }
  __syncthreads();
  if (part == 0) {
    const auto sum = [&](int g) { return acc.group(g) + meet[g * 64]; };
    quadrant_image<F, false>(sum, scale, images + quadrant * F::kImageBytes, L);
    if (kept != nullptr) {
      const int p = quadrant >> 1, q = quadrant & 1;
#pragma unroll
      for (int g = 0; g < F::Acc::kGroups; ++g) {
        const f32x4_t v = sum(g);
        const int row = p * Dh + F::Acc::group_row(g, L), col = q * Dh + F::Acc::group_col(g, L);
#pragma unroll
        for (int i = 0; i < 4; ++i) kept[(row + i) * D + col] = v[i];
      }
    }
  }
  __syncthreads();
}

template <class F>
__global__ __launch_bounds__(512) void wide_fused_fwd_kernel(const LaunchArgs a, float* __restrict__ kept) {
  using Lds = FusedLds<F, 1>;
  constexpr int Dh = F::D, D = 2 * Dh;
  const Lane L;
  const int bh = blockIdx.x;
  const size_t base = a.st.slice_base(bh, a.H);
  unsigned char* images = smem;
  unsigned char* sets = smem + Lds::kTiles;
  typename F::Acc acc;
  {
    const WideSrc kv(a.K + base, a.V + base, a.N, a.st.row.stride);
    const uint8_t* keys = a.mask == nullptr ? nullptr : a.mask + static_cast<size_t>(bh / a.H) * a.N;
    fused_state_pass<F, Lds::kWaveBytes>(acc, kv, keys, a.N, L.wave * TR, 8 * TR, a.eps, sets, L);
  }
  const float scale = a.slice_scale != nullptr ? a.slice_scale[bh] : a.scale;
  ApplyArgs r{};
  r.X = a.Q + base;
  r.mask = nullptr;  // queries are not masked
  r.out = a.O + base;
  r.N = a.N;
  r.r_begin = 0;
  r.r_end = a.N;
  r.stride = a.st.row.stride;
  r.scale = scale;
  r.eps = a.eps;
  // the first tile of Q travels while the images are made
  WideRaw first;
  request_first_tile<8>(first, r, L);
  forward_images<F>(acc, scale, images, sets, kept == nullptr ? nullptr : kept + static_cast<size_t>(bh) * D * D, L);
  plain_tiles<F, 8, true, true>(r, images, sets + L.wave * Lds::kWaveBytes, L, &first);
}

// A group of four waves owns its slice completely: one quadrant of the state per wave, rounds of 64 rows, no sums
// to meet.  `rows`: N, or 0 where the group has no slice and only keeps step.
template <class F>
__device__ __forceinline__ void owned_slice_fwd(const LaunchArgs& a, int bh, int rows, unsigned char* images,
                                                unsigned char* sets, float* __restrict__ kept, const Lane& L) {
  constexpr int kWaveBytes = FusedLds<F, 1>::kWaveBytes, Dh = F::D, D = 2 * Dh;
  const int quadrant = L.wave & 3;
  const size_t base = a.st.slice_base(bh, a.H);
  typename F::Acc acc;
  {
    const WideSrc kv(a.K + base, a.V + base, a.N, a.st.row.stride);
    const uint8_t* keys = a.mask == nullptr ? nullptr : a.mask + static_cast<size_t>(bh / a.H) * a.N;
    fused_state_pass<F, kWaveBytes>(acc, kv, keys, a.N, quadrant * TR, 4 * TR, a.eps, sets, L, false, rows);
  }
  const float scale = a.slice_scale != nullptr ? a.slice_scale[bh] : a.scale;
  Lane Lg = L;  // the wave's place in its group
  Lg.wave = quadrant;
  ApplyArgs r{};
  r.X = a.Q + base;
  r.mask = nullptr;  // queries are not masked
  r.out = a.O + base;
  r.N = a.N;
  r.r_begin = 0;
  r.r_end = rows;
  r.stride = a.st.row.stride;
  r.scale = scale;
  r.eps = a.eps;
  WideRaw first;
  request_first_tile<4>(first, r, Lg);
  const auto own = [&](int g) { return acc.group(g); };
  quadrant_image<F, false>(own, scale, images + quadrant * F::kImageBytes, L);
  if (kept != nullptr && rows > 0) {  // S as it is, row-major, for the caller's backward call
    float* __restrict__ out = kept + static_cast<size_t>(bh) * D * D;
    const int p = quadrant >> 1, q = quadrant & 1;
#pragma unroll
    for (int g = 0; g < F::Acc::kGroups; ++g) {
      const f32x4_t v = acc.group(g);
      const int row = p * Dh + F::Acc::group_row(g, L), col = q * Dh + F::Acc::group_col(g, L);
#pragma unroll
      for (int i = 0; i < 4; ++i) out[(row + i) * D + col] = v[i];
    }
  }
  __syncthreads();
  plain_tiles<F, 4, true, true>(r, images, sets + L.wave * kWaveBytes, Lg, &first);
}

// The forward with a workgroup of four waves per slice, two of them on a compute unit, each slice at a pace of its own.
template <class F>
__global__ __launch_bounds__(256, 2) void wide_small_fwd_kernel(const LaunchArgs a, float* __restrict__ kept) {
  owned_slice_fwd<F>(a, blockIdx.x, a.N, smem, smem + FusedLds<F, 1, 4>::kTiles, kept, Lane());
}

// The forward with two slices per workgroup (waves 0-3 one slice, waves 4-7 the next), which share the barriers.
template <class F>
__global__ __launch_bounds__(512) void wide_paired_fwd_kernel(const LaunchArgs a, int slices,
                                                              float* __restrict__ kept) {
  using Lds = FusedLds<F, 2>;
  const Lane L;
  const int group = L.wave >> 2, slice = 2 * blockIdx.x + group;
  const bool exists = slice < slices;
  owned_slice_fwd<F>(a, exists ? slice : 0, exists ? a.N : 0, smem + group * Lds::kSetBytes, smem + Lds::kTiles, kept,
                     L);
}

// d loss / d log(scale) = scale <S, dS> of the slice: the dS accumulators (waves 4-7) meet the S
// accumulators (waves 0-3) in `area` (free at that point), the sum in a fixed order.  Ends with
// a barrier.
template <class F>
__device__ __forceinline__ void state_dot(const typename F::Acc& acc, bool second, float scale,
                                          unsigned char* area, float* __restrict__ out, const Lane& L) {
  const int quadrant = L.wave & 3;
  f32x4_t* meet = reinterpret_cast<f32x4_t*>(area) + quadrant * F::Acc::kGroups * 64 + L.lane;
  float* partial = reinterpret_cast<float*>(area + 4 * F::Acc::kGroups * 64 * 16);
  if (second) {
#pragma unroll
    for (int g = 0; g < F::Acc::kGroups; ++g) meet[g * 64] = acc.group(g);
  }
  __syncthreads();
  if (!second) {
    float dot = 0.0f;
#pragma unroll
    for (int g = 0; g < F::Acc::kGroups; ++g) {
      const f32x4_t s = acc.group(g), d = meet[g * 64];
#pragma unroll
      for (int i = 0; i < 4; ++i) dot += s[i] * d[i];
    }
    dot = wave_sum(dot);
    if (L.lane == 0) partial[quadrant] = dot;
  }
  __syncthreads();
  if (threadIdx.x == 0) *out = (((partial[0] + partial[1]) + partial[2]) + partial[3]) * scale;
  __syncthreads();  // the area is written again next
}

template <class F>
__global__ __launch_bounds__(512) void wide_fused_bwd_kernel(const LaunchArgs a, float* __restrict__ dlog) {
  using Lds = FusedLds<F, 2>;
  const Lane L;
  const int bh = blockIdx.x;
  const size_t base = a.st.slice_base(bh, a.H);
  unsigned char* images_a = smem;                    // S natural, later dS natural
  unsigned char* images_b = smem + Lds::kSetBytes;   // dS transposed
  unsigned char* sets = smem + Lds::kTiles;
  const int quadrant = L.wave & 3;
  const bool second = L.wave >= 4;  // waves 4-7: dS = sum_i qhat_i^T dO_i
  const uint8_t* keys = a.mask == nullptr ? nullptr : a.mask + static_cast<size_t>(bh / a.H) * a.N;
  // S is needed as natural images only: its waves sum up the transposed quadrants, unless the
  // accumulators of S and dS are to meet lane by lane for <S, dS>
  const bool swapped = !second && dlog == nullptr;
  typename F::Acc acc;
  {
    const WideSrc src((second ? a.Q : a.K) + base, (second ? a.dO : a.V) + base, a.N, a.st.row.stride);
    fused_state_pass<F, Lds::kWaveBytes>(acc, src, second ? nullptr : keys, a.N, quadrant * TR, 4 * TR,
                                         a.eps, sets, L, swapped);
  }
  const float scale = a.slice_scale != nullptr ? a.slice_scale[bh] : a.scale;
  const auto own = [&](int g) { return acc.group(g); };
  if (dlog != nullptr) state_dot<F>(acc, second, scale, sets, dlog + bh, L);
  if (swapped) quadrant_image<F, false>(own, scale, images_a + quadrant * F::kImageBytes, L);
  else if (!second) quadrant_image<F, true>(own, scale, images_a + quadrant * F::kImageBytes, L);
  else quadrant_image<F, false>(own, scale, images_b + quadrant * F::kImageBytes, L);
  __syncthreads();

  unsigned char* tiles = sets + L.wave * Lds::kWaveBytes;
  ApplyArgs r{};
  r.N = a.N;
  r.r_begin = 0;
  r.r_end = a.N;
  r.stride = a.st.row.stride;
  r.scale = scale;
  r.eps = a.eps;
  // dQ
  r.X = a.Q + base;
  r.Y = a.dO + base;
  r.mask = nullptr;
  r.out = a.dQ + base;
  projected_tiles<F, 8>(r, images_a, tiles, L);
  __syncthreads();  // nobody reads the images of S any more
  if (second) quadrant_image<F, true>(own, scale, images_a + quadrant * F::kImageBytes, L);
  // dV
  r.X = a.K + base;
  r.mask = keys;
  r.out = a.dV + base;
  plain_tiles<F, 8, false>(r, images_b, tiles, L);
  __syncthreads();  // the natural images of dS are complete
  // dK
  r.Y = a.V + base;
  r.out = a.dK + base;
  projected_tiles<F, 8>(r, images_a, tiles, L);
}

// ---- short sequences (N <= 256), backward: every tile requested at once and kept in registers -----
//
// The backward for sequences of at most 256 rows: a wave asks for all its rows at the start
// (everything the slice needs is in flight together) and keeps them in registers, so the apply
// roles read nothing again.  Waves 0-3, which hold rows of (K, V), compute dV and dK for them and
// waves 4-7, which hold rows of (Q, dO), dQ; all three image sets are written as soon as the states are
// complete (LDS: [S natural | dS natural | dS transposed], and over the same memory the two round buffers
// of the state phase).  A wave holds 32 consecutive rows at a time, 16 staged per round; when both halves are
// staged it reads them back as it needs them for products over 32 rows (xhat and y, 16 of every 32 bytes of
// a row): these take half the operand reads of products over 16, and nothing is staged or normalised again.
//
// Bound by what follows one another in a workgroup (one per compute unit): the first rows' way from memory, the states, the
// images, the products, the stores.  us, products over 16 rows staged again and this, bf16, left-padded lengths uniform in 0 ... N, over
// the same buffers: 1024 slices x 200 rows 78.8, 75.1 (fresh ones 80.6, 3.9 TB/s); 512 x 100 24.9, 20.9; 300 x 256 41.5, 39.6; 90 x 200
// 19.3, 16.0; 1024 x 50 33.5, 28.3; ELU + 1, 512 x 200 49.8, 42.5.  Traffic: each row once (256 x 200: 39.1 MB fetched, 39.3 written).
constexpr int kKeptRows = 256;
// Sequences of so many rounds of 64 rows: a workgroup takes one slice after the other, the next one's rows requested ahead.  Longer
// ones leave no registers for that (fresh buffers, 1024 x 50 rows 35.0 without, 31.2; two rounds, 1024 x 128: 47.1 without, 49.5; four, 300 x 256: 42.2, 47.2).
constexpr int kAheadRounds = 1;

template <class F>
struct KeptLds {
  static constexpr int kSetBytes = 4 * F::kImageBytes;
  static constexpr int kRoundWave = 4 * kTileBytes;  // state phase: two round buffers from offset 0
  static constexpr int kRoundBuffer = 8 * kRoundWave;
  static constexpr int kBytes = 3 * kSetBytes > 2 * kRoundBuffer ? 3 * kSetBytes : 2 * kRoundBuffer;
  static_assert(4 * F::Acc::kGroups * 64 * 16 + 64 <= kBytes, "accumulators meet in the same memory");
};

// 32 rows of a tensor pair in the layout of products over 32 rows: chunk c is bytes 32 c + 16 half .. + 15 of row
// lane%32, half = lane/32.
template <class F>
struct Rows32 {
  typename F::v8_t x[8], y[8];
  float inv;  // 1/r, -0: the row does not take part
};

// The two staged tiles of a wave (`first`: rows 0-15, `second`: rows 16-31, each [xhat pieces | y pieces] with 1/r in
// the padding of the first piece's rows).
template <class F>
__device__ __forceinline__ void fetch_rows32(Rows32<F>& t, const unsigned char* first, const unsigned char* second,
                                             bool has_second, const Lane& L) {
  const unsigned char* at = ((L.lane & 16) != 0 && has_second ? second : first) + L.i16 * kTileStride;
  const int half = 16 * (L.lane >> 5);
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const unsigned char* piece = at + (c >> 2) * kTileBytes + 32 * (c & 3) + half;
    t.x[c] = *reinterpret_cast<const typename F::v8_t*>(piece);
    t.y[c] = *reinterpret_cast<const typename F::v8_t*>(piece + P * kTileBytes);
  }
  t.inv = *reinterpret_cast<const float*>(at + kRowBytes);
}

// The state phase over tiles already in registers (see fused_state_pass).  Two round buffers take turns: the tiles of the
// next round are staged while those of this one are added up, one barrier per round.  Ends with a barrier (the
// buffers are free).  An odd number of rounds: the last rows are 16, twice.
template <class F, int ROUNDS>
__device__ __forceinline__ void kept_state_pass(typename F::Acc& acc, const WideRaw (&kept)[ROUNDS],
                                                Rows32<F> (&rows)[(ROUNDS + 1) / 2], float eps, const Lane& L0,
                                                bool swapped) {
  constexpr int kRoundWave = KeptLds<F>::kRoundWave, kSecond = KeptLds<F>::kRoundBuffer;
  const int quadrant = L0.wave & 3, p = quadrant >> 1, q = quadrant & 1, group = L0.wave >> 2;
  const int left = (swapped ? 2 + q : p) * kTileBytes, right = (swapped ? p : 2 + q) * kTileBytes;
  unsigned char* mine = smem + L0.wave * kRoundWave;
  const auto stage = [&](int r) {
    const Lane L = L0.again();
    float inv[2];
    unsigned char* tiles = mine + (r & 1) * kSecond;
    stage_wide<F, mapped_mode<F>(), true, true>(kept[r], L, eps, tiles, inv);
    if (L.ch == 0) {
#pragma unroll
      for (int h = 0; h < 2; ++h) *reinterpret_cast<float*>(tiles + (L.r8 + 8 * h) * kTileStride + kRowBytes) = inv[h];
    }
  };
  acc.zero();
  stage(0);
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    __syncthreads();  // round r is staged; nobody reads the other buffer any more
    const Lane L = L0.again();
    if ((r & 1) != 0 || r + 1 == ROUNDS) {  // (the wave's own tiles: written before the barrier)
      Rows32<F>& t = rows[r / 2];
      fetch_rows32<F>(t, mine, mine + kSecond, (r & 1) != 0, L);
      wave_lds_fence();
    }
    if (r + 1 < ROUNDS) stage(r + 1 < ROUNDS ? r + 1 : 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const unsigned char* tile = smem + (r & 1) * kSecond + (4 * group + t) * kRoundWave;
      acc.mfma(tile + left, tile + right, L);
    }
  }
  __syncthreads();
}

// Block nb of the rows (values 8 t .. of a lane: 16 bytes at 64 nb + 32 t + 16 half of its row).  The lanes of rows 0-15
// and 16-31 exchange chunks first, so that a store writes 64 contiguous bytes of each of 16 rows: with 32 of
// each of 32 the streamed stores reach memory as parts of lines (1024 slices x 200 rows, backward: 220 us).
struct StoreRows32 {
  __amdgpu_buffer_rsrc_t out;  // ends with row end - 1: rows beyond are dropped without a branch
  uint32_t at;                 // of the first store: row lane%16, bytes 32 (group & 1) + 16 (group / 2)
  int stride;
  __device__ __forceinline__ StoreRows32(unsigned char* base, int row0, int end, int stride_bytes, const Lane& L)
      : out(__builtin_amdgcn_make_buffer_rsrc(base, 0, end > row0 ? (end - 1) * stride_bytes + P * kHalfBytes : 0, 0x00020000)),
        at(static_cast<uint32_t>(row0 + L.i16) * stride_bytes + 32 * (L.g16 & 1) + 16 * (L.g16 >> 1)),
        stride(stride_bytes) {}
  template <class F>
  __device__ __forceinline__ void store(int nb, const f32x16_t& v) const {
    u32x4_t t[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      float f[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = v[8 * k + i];
      t[k] = F::pack(f);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const auto swapped = __builtin_amdgcn_permlane16_swap(t[0][i], t[1][i], false, false);
      t[0][i] = swapped[0];
      t[1][i] = swapped[1];
    }
    __builtin_amdgcn_raw_buffer_store_b128(t[0], out, at + 64 * nb, 0, kStoreStreamed);
    __builtin_amdgcn_raw_buffer_store_b128(t[1], out, at + 16 * stride + 64 * nb, 0, kStoreStreamed);
  }
};

// Zeros over some of 32 rows (bit i: row row0 + i), four lanes a row.
__device__ __forceinline__ void zero_rows32(unsigned char* base, int row0, int end, int stride, uint32_t rows, const Lane& L) {
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = 16 * k + L.i16;
    if (((rows >> i) & 1) == 0 || row0 + i >= end) continue;
    u32x4_t* at = reinterpret_cast<u32x4_t*>(base + static_cast<size_t>(row0 + i) * stride) + L.g16;
#pragma unroll
    for (int c = 0; c < 4; ++c) at[4 * c] = u32x4_t{0, 0, 0, 0};
  }
}

// Blocks 0 and 1 of a half row of the product of 32 rows X with the images first, first + step: sum over the halves of X.
// (Two chains of products that wait for themselves only.)
template <class F>
__device__ __forceinline__ void blocks32(const typename F::v8_t (&X)[8], const unsigned char* images, int first,
                                         int step, const Lane& L, f32x16_t& v0, f32x16_t& v1) {
#pragma unroll
  for (int i = 0; i < 16; ++i) v0[i] = v1[i] = 0.0f;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const unsigned char* image = images + (first + (c >> 2) * step) * F::kImageBytes;
    v0 = F::Elem::mfma32(F::operand32(image, 0, c & 3, L), X[c], v0);
    v1 = F::Elem::mfma32(F::operand32(image, 1, c & 3, L), X[c], v1);
  }
}

// 32 kept rows in the backward: (K rows only) dV = khat (scale dS), then g = y (natural images)^T and
// out = (g - xhat (xhat . g)) / r.
template <class F>
__device__ __forceinline__ void kept_rows_bwd(Rows32<F>& t, int row0, int end, bool plain_too,
                                              const unsigned char* natural, const unsigned char* transposed,
                                              unsigned char* out_projected, unsigned char* out_plain, int stride,
                                              const Lane& L) {
  const StoreRows32 projected(out_projected, row0, end, stride, L), plain(out_plain, row0, end, stride, L);
  const uint32_t masked = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(is_masked(t.inv)));  // (absent rows too)
  if (masked == ~0u) {  // zeros
    f32x16_t z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.0f;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      if (plain_too) plain.store<F>(nb, z);
      projected.store<F>(nb, z);
    }
    return;
  }
  if (plain_too) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      f32x16_t o[2];
      blocks32<F>(t.x, transposed, q, 2, L, o[0], o[1]);
      plain.store<F>(2 * q, o[0]);
      plain.store<F>(2 * q + 1, o[1]);
    }
  }
  f32x16_t g[4];
#pragma unroll
  for (int p = 0; p < 2; ++p) blocks32<F>(t.y, natural, 2 * p, 1, L, g[2 * p], g[2 * p + 1]);
  const auto unit = [&](int c, float (&u)[8]) { F::unpack(__builtin_bit_cast(u32x4_t, t.x[c]), u); };
  float check = 0.0f;  // masked rows: 0 if the state is finite, NaN if not
  if (F::kMap == kMapElu1) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      float u[8];
      unit(c, u);
#pragma unroll
      for (int i = 0; i < 8; ++i) g[c >> 1][8 * (c & 1) + i] *= fminf(u[i], 1.0f);
    }
    if (masked != 0) {
#pragma unroll
      for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int i = 0; i < 16; ++i) check += g[nb][i];
    }
  } else {
    float proj = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      float u[8];
      unit(c, u);
#pragma unroll
      for (int i = 0; i < 8; ++i) proj += u[i] * g[c >> 1][8 * (c & 1) + i];
    }
    proj += __shfl_xor(proj, 32);
    check = proj;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      u32x4_t again = __builtin_bit_cast(u32x4_t, t.x[c]);  // (unpacked again rather than kept: 64 registers)
      asm volatile("" : "+v"(again));
      float u[8];
      F::unpack(again, u);
#pragma unroll
      for (int i = 0; i < 8; ++i)  // (1/r of masked rows is -0: the sign would reach their zeros)
        g[c >> 1][8 * (c & 1) + i] = (g[c >> 1][8 * (c & 1) + i] - u[i] * proj) * fabsf(t.inv);
    }
  }
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) projected.store<F>(nb, g[nb]);
  // Masked rows are zeros as products of zero rows, but NaN where a value of the state is not finite.  That value is in the
  // sums of g of every row, and so in `check`: then zeros go over them, which costs the others nothing.
  const uint64_t not_zero = __builtin_amdgcn_ballot_w64(is_masked(t.inv) && !(check == 0.0f));  // (ELU + 1: each lane of its half row)
  if (not_zero != 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (behind the stores above)
    zero_rows32(out_projected, row0, end, stride, static_cast<uint32_t>(not_zero | not_zero >> 32), L);
    if (plain_too) zero_rows32(out_plain, row0, end, stride, static_cast<uint32_t>(not_zero | not_zero >> 32), L);
  }
}

// For sequences of ROUNDS rounds of 64 rows.  A workgroup takes slices blockIdx.x, + gridDim.x, ... (ROUNDS <= kAheadRounds; the
// others one), the rows of the next one requested when this one's are no longer needed.  (No branch around
// loads or rounds: what is held would no longer fit the registers.)
template <class F, int ROUNDS>
__global__ __launch_bounds__(512) void wide_kept_bwd_kernel(const LaunchArgs a, int slices, float* __restrict__ dlog) {
  using Lds = KeptLds<F>;
  constexpr int kPairs = (ROUNDS + 1) / 2;
  constexpr bool kAhead = ROUNDS <= kAheadRounds;
  const Lane L0;
  const int stride = a.st.row.stride, N = a.N;
  const int quadrant = L0.wave & 3;
  const bool second = L0.wave >= 4;  // waves 4-7: (Q, dO) rows, dS = sum_i qhat_i^T dO_i, dQ
  // Which 32 of 128 rows the wave holds (16, and one round for all of them, where 64 or fewer are left): the two waves of a
  // SIMD (w and w + 4) take different ones, so that a ragged end does not leave both with more rows than the rest
  const int slot = second ? (quadrant + 2) & 3 : quadrant;
  const auto rows_of = [&](int j) { return 2 * j + 1 < ROUNDS ? 32 : TR; };
  const auto first_of = [&](int j) { return 128 * j + rows_of(j) * slot; };
  const auto first_of_round = [&](int r) { return first_of(r / 2) + TR * (r & 1); };
  // the key mask's bytes of the lane's rows, requested long before the rows
  const bool masked = !second && a.mask != nullptr;
  struct KeyBytes {
    unsigned of[ROUNDS][2];
  };
  const auto request_keys = [&](int bh, const Lane& L) {
    const auto keys = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(a.mask) + (masked ? static_cast<size_t>(bh / a.H) * N : 0), 0, masked ? N : 0, 0x00020000);
    KeyBytes b;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        b.of[r][h] = __builtin_amdgcn_raw_buffer_load_b8(keys, first_of_round(r) + L.r8 + 8 * h, 0, 0);
    return b;
  };
  const auto request = [&](WideRaw& t, const WideSrc& src, const KeyBytes& b, int r, const Lane& L) {
    const int row0 = first_of_round(r);
    int bits = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      bits |= static_cast<int>(row0 + L.r8 + 8 * h < N && (!masked || b.of[r][h] != 0)) << h;
    load_wide<true>(t, L, src, row0, bits);
  };
  const auto source = [&](int bh, int n) {  // n = 0: nothing is fetched
    const size_t base = a.st.slice_base(bh, a.H);
    return WideSrc((second ? a.Q : a.K) + base, (second ? a.dO : a.V) + base, n, stride);
  };
  // S is needed as natural images only: its waves sum up the transposed quadrants, unless the
  // accumulators of S and dS are to meet lane by lane for <S, dS>
  const bool swapped = !second && dlog == nullptr;

  WideRaw kept[ROUNDS];
  int bh = blockIdx.x;
  {
    // (each masked tile behind the bytes that decide on it, and these behind the tile before: what is needed first comes first)
    const WideSrc src = source(bh, N);
    const uint8_t* m = masked ? a.mask + static_cast<size_t>(bh / a.H) * N : nullptr;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) load_wide<true>(kept[r], L0, src, first_of_round(r), row_bits(m, first_of_round(r), N, L0));
  }
#pragma unroll 1
  while (true) {
    const int next = bh + static_cast<int>(gridDim.x);
    const bool more = next < slices;
    typename F::Acc acc;
    Rows32<F> rows[kPairs];
    kept_state_pass<F, ROUNDS>(acc, kept, rows, a.eps, L0, swapped);
    const Lane L = L0.again();
    KeyBytes next_keys;
    if (kAhead) next_keys = request_keys(more ? next : bh, L);
    const float scale = a.slice_scale != nullptr ? a.slice_scale[bh] : a.scale;
    if (dlog != nullptr) state_dot<F>(acc, second, scale, smem, dlog + bh, L);
    typedef typename F::Image32 Image;
    const auto own = [&](int g) { return acc.group(g); };
    if (swapped) {
      quadrant_image<F, false, Image>(own, scale, smem + quadrant * F::kImageBytes, L);
    } else if (!second) {
      quadrant_image<F, true, Image>(own, scale, smem + quadrant * F::kImageBytes, L);
    } else {
      quadrant_image<F, true, Image>(own, scale, smem + Lds::kSetBytes + quadrant * F::kImageBytes, L);
      quadrant_image<F, false, Image>(own, scale, smem + 2 * Lds::kSetBytes + quadrant * F::kImageBytes, L);
    }
    __syncthreads();
    const size_t base = a.st.slice_base(bh, a.H);
    unsigned char* out_projected = (second ? a.dQ : a.dK) + base;
    const WideSrc src = source(more ? next : bh, more ? N : 0);
    // (opaque: as constants they would be added to every address, the sets lying beyond the 64 KB that an LDS read can add)
    int natural_at = second ? 0 : Lds::kSetBytes, transposed_at = 2 * Lds::kSetBytes;
    asm volatile("" : "+s"(natural_at), "+s"(transposed_at));
    const unsigned char *natural = smem + natural_at, *transposed = smem + transposed_at;
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
      const Lane L = L0.again();
      const int row0 = first_of(j), end = row0 + rows_of(j) < N ? row0 + rows_of(j) : N;
      if (row0 < N)
        kept_rows_bwd<F>(rows[j], row0, end, !second, natural, transposed, out_projected, a.dV + base, stride, L);
#pragma unroll
      for (int r = 2 * j; kAhead && r < 2 * j + 2 && r < ROUNDS; ++r) request(kept[r], src, next_keys, r, L);
    }
    if (!kAhead || !more) break;
    bh = next;
    __syncthreads();  // the images are written over next
  }
}

// ---- host side ------------------------------------------------------------------------------------

Strides byte_strides(const Problem& p) {
  return Strides{p.stride_batch * p.elem_bytes(), p.stride_head * p.elem_bytes(),
                 RowAddr{static_cast<int>(p.stride_row * p.elem_bytes()),
                         static_cast<int>(p.D * p.elem_bytes())}};
}

LaunchArgs launch_args(const Problem& p, const Plan& plan, const float* states, const float* dstates) {
  LaunchArgs a{};
  a.Q = static_cast<const unsigned char*>(p.Q);
  a.K = static_cast<const unsigned char*>(p.K);
  a.V = static_cast<const unsigned char*>(p.V);
  a.dO = static_cast<const unsigned char*>(p.dO);
  a.mask = p.mask;
  a.states = states;
  a.dstates = dstates;
  a.O = static_cast<unsigned char*>(p.O);
  a.dQ = static_cast<unsigned char*>(p.dQ);
  a.dK = static_cast<unsigned char*>(p.dK);
  a.dV = static_cast<unsigned char*>(p.dV);
  a.H = p.H;
  a.N = p.N;
  a.splits = plan.splits;
  a.rows_per_split = plan.rows_per_split;
  a.scale = p.scale;
  a.eps = p.eps;
  a.slice_scale = p.slice_scale;
  a.st = byte_strides(p);
  return a;
}

// Workgroups of 8 waves (the whole LDS of a compute unit at their disposal) when the launch has
// no more workgroups than there are compute units, of 4 waves (two per compute unit) otherwise.
constexpr int kUnits = 256;
template <int WAVES>
constexpr int max_lds_bytes() {
  return WAVES == 8 ? 160 * 1024 : 80 * 1024;
}

template <class F, int WAVES>
hipError_t states_w(const Problem& p, const Plan& plan, bool bwd) {
  constexpr int D = P * F::D;
  constexpr int lds = WAVES * 2 * P * kTileBytes;
  static_assert(lds <= max_lds_bytes<WAVES>(), "round buffer");
  const unsigned blocks = static_cast<unsigned>(p.B) * p.H * plan.splits;
  const size_t second = static_cast<size_t>(blocks) * D * D;
  const hipError_t err = grant_dynamic_lds(reinterpret_cast<const void*>(wide_state_kernel<F, WAVES>),
                                           max_lds_bytes<WAVES>());
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL((wide_state_kernel<F, WAVES>), dim3(blocks, bwd ? 2 : 1), dim3(64 * WAVES), lds,
                     p.stream, static_cast<const unsigned char*>(p.Q),
                     static_cast<const unsigned char*>(p.K), static_cast<const unsigned char*>(p.V),
                     static_cast<const unsigned char*>(p.dO), p.mask, p.workspace, p.H, p.N,
                     plan.splits, bwd ? plan.rows_per_split : 0, second, p.eps, byte_strides(p));
  return hipGetLastError();
}

template <class F, int WAVES>
hipError_t apply_w(const Problem& p, const Plan& plan, const float* st, const float* dst, bool bwd) {
  constexpr int lds = ApplyLds<F, WAVES>::kBytes;
  static_assert(lds <= max_lds_bytes<WAVES>(), "images and tiles");
  const LaunchArgs a = launch_args(p, plan, st, dst);
  const unsigned blocks = static_cast<unsigned>(p.B) * p.H * plan.splits;
  const void* kern = bwd ? reinterpret_cast<const void*>(wide_bwd_kernel<F, WAVES>)
                         : reinterpret_cast<const void*>(wide_fwd_kernel<F, WAVES>);
  const hipError_t err = grant_dynamic_lds(kern, max_lds_bytes<WAVES>());
  if (err != hipSuccess) return err;
  if (bwd)
    hipLaunchKernelGGL((wide_bwd_kernel<F, WAVES>), dim3(blocks, 3), dim3(64 * WAVES), lds, p.stream, a);
  else
    hipLaunchKernelGGL((wide_fwd_kernel<F, WAVES>), dim3(blocks), dim3(64 * WAVES), lds, p.stream, a);
  return hipGetLastError();
}

// `kinds`: workgroups per (slice, split) of the launch (states or roles)
inline bool few_workgroups(const Problem& p, const Plan& plan, int kinds) {
  return static_cast<long>(p.B) * p.H * plan.splits * kinds <= kUnits;
}

template <class F>
hipError_t states(const Problem& p, const Plan& plan, bool bwd) {
  return few_workgroups(p, plan, bwd ? 2 : 1) ? states_w<F, 8>(p, plan, bwd)
                                              : states_w<F, 4>(p, plan, bwd);
}

template <class F>
hipError_t apply(const Problem& p, const Plan& plan, const float* st, const float* dst, bool bwd) {
  return few_workgroups(p, plan, bwd ? 3 : 1) ? apply_w<F, 8>(p, plan, st, dst, bwd)
                                              : apply_w<F, 4>(p, plan, st, dst, bwd);
}

template <class F>
hipError_t fused(const Problem& p, const Plan& plan, bool bwd) {
  static_assert(FusedLds<F, 2>::kBytes <= max_lds_bytes<8>(), "two image sets and the tile sets");
  constexpr int lds_fwd = FusedLds<F, 1>::kBytes, lds_bwd = FusedLds<F, 2>::kBytes;
  const LaunchArgs a = launch_args(p, plan, nullptr, nullptr);
  const unsigned blocks = static_cast<unsigned>(p.B) * p.H;
  if (bwd && p.N <= kKeptRows) {
    constexpr int lds_kept = KeptLds<F>::kBytes;
    static_assert(lds_kept <= max_lds_bytes<8>(), "three image sets, two round buffers");
    const auto launch = [&](auto kernel) {
      const hipError_t err = grant_dynamic_lds(reinterpret_cast<const void*>(kernel), max_lds_bytes<8>());
      if (err != hipSuccess) return err;
      hipLaunchKernelGGL(kernel, dim3(p.N <= 4 * TR * kAheadRounds && blocks > kUnits ? kUnits : blocks), dim3(512), lds_kept, p.stream, a,
                         static_cast<int>(blocks), p.dlog_scale);
      return hipGetLastError();
    };
    switch ((p.N - 1) / (4 * TR)) {
      case 0: return launch(wide_kept_bwd_kernel<F, 1>);
      case 1: return launch(wide_kept_bwd_kernel<F, 2>);
      case 2: return launch(wide_kept_bwd_kernel<F, 3>);
      default: return launch(wide_kept_bwd_kernel<F, 4>);
    }
  }
  const void* kern = bwd ? reinterpret_cast<const void*>(wide_fused_bwd_kernel<F>)
                         : reinterpret_cast<const void*>(wide_fused_fwd_kernel<F>);
  const hipError_t err = grant_dynamic_lds(kern, max_lds_bytes<8>());
  if (err != hipSuccess) return err;
  // Forward, more slices than compute units: four waves per slice.  A workgroup each while all of them run at once (in pairs,
  // 260 slices would leave every other compute unit idle) or the sequences are a round of 64 rows at most, pairs in
  // one workgroup beyond.  us, pairs and one each, bf16: 260 x 200 rows 17.5, 15.2;  300 x 200 18.1, 16.5;  512 x 100 11.1, 10.8;
  // 2048 x 20 20.5, 19.0;  1024 x 50 12.8, 12.4;  1024 x 200 35.8, 37.3.
  if (!bwd && blocks > static_cast<unsigned>(kUnits)) {
    constexpr int lds_small = FusedLds<F, 1, 4>::kBytes;
    static_assert(lds_small <= max_lds_bytes<4>(), "two workgroups per compute unit");
    const bool small = blocks <= static_cast<unsigned>(2 * kUnits) || p.N <= 64;
    const hipError_t e2 =
        small ? grant_dynamic_lds(reinterpret_cast<const void*>(wide_small_fwd_kernel<F>), max_lds_bytes<4>())
              : grant_dynamic_lds(reinterpret_cast<const void*>(wide_paired_fwd_kernel<F>), max_lds_bytes<8>());
    if (e2 != hipSuccess) return e2;
    if (small)
      hipLaunchKernelGGL((wide_small_fwd_kernel<F>), dim3(blocks), dim3(256), lds_small, p.stream, a, p.saved_state);
    else
      hipLaunchKernelGGL((wide_paired_fwd_kernel<F>), dim3((blocks + 1) / 2), dim3(512), lds_bwd, p.stream, a,
                         static_cast<int>(blocks), p.saved_state);
    return hipGetLastError();
  }
  if (bwd)
    hipLaunchKernelGGL((wide_fused_bwd_kernel<F>), dim3(blocks), dim3(512), lds_bwd,
                       p.stream, a, p.dlog_scale);
  else
    hipLaunchKernelGGL((wide_fused_fwd_kernel<F>), dim3(blocks), dim3(512), lds_fwd,
                       p.stream, a, p.saved_state);
  return hipGetLastError();
}

}  // namespace wide
}  // namespace

bool wide_supports(int dtype, int D) { return dtype == 0 ? (D == 64 || D == 128) : D == 128; }

namespace {
// fn(F{}) for the element format of the problem (16-bit), with the feature map of its params
template <class Fn>
hipError_t for_format(const Problem& p, Fn fn) {
  using namespace mfma;
  if (p.feature_map == kMapElu1) return p.dtype == 1 ? fn(WithElu1<Bf16x64>{}) : fn(WithElu1<F16x64>{});
  return p.dtype == 1 ? fn(Bf16x64{}) : fn(F16x64{});
}
}  // namespace

hipError_t launch_wide_states(const Problem& p, const Plan& plan, bool bwd) {
  if (p.dtype == 0) return launch_wide32_states(p, plan, bwd);
  return for_format(p, [&](auto f) { return wide::states<decltype(f)>(p, plan, bwd); });
}

// One launch per direction whenever the sequence is not cut - except, with 16-bit rows, a backward
// over so few slices that its three roles as workgroups of their own are what fills the chip (64
// slices of 200 rows, bf16 d_h = 128: 17.5 us against 19.4 us in one launch; the forward: 13.8
// against 10.0).
bool wide_fused_applies(int dtype, int B, int H, int splits, bool bwd) {
  return splits == 1 && !(dtype != 0 && bwd && static_cast<long>(B) * H * 3 <= wide::kUnits);
}

hipError_t launch_wide_fused(const Problem& p, const Plan& plan, bool bwd) {
  if (!wide_fused_applies(p.dtype, p.B, p.H, plan.splits, bwd)) return hipErrorInvalidValue;
  if (columns_apply(p, bwd)) return launch_columns(p, bwd);
  if (p.dtype == 0) return launch_wide32_fused(p, plan, bwd);
  return for_format(p, [&](auto f) { return wide::fused<decltype(f)>(p, plan, bwd); });
}

hipError_t launch_wide_apply(const Problem& p, const Plan& plan, const float* states,
                             const float* dstates, bool bwd) {
  if (p.dtype == 0) return launch_wide32_apply(p, plan, states, dstates, bwd);
  return for_format(p, [&](auto f) { return wide::apply<decltype(f)>(p, plan, states, dstates, bwd); });
}

}  // namespace cotten
