// Resident kernels for short sequences of 16-bit elements (bf16 or fp16, N <= 208, d_h = 64); up to 128 rows: short_*_kernel.
//
// One persistent workgroup of 16 waves owns one slice at a time and keeps it in LDS: wave w
// loads and stages the 16-row tile w, so every global load of the slice is issued at once and
// nothing is read twice; the loads of the workgroup's next slice are issued as soon as the
// registers are free and travel while the current slice is worked on.  The d x d states are
// built by one wave per output block, each walking all resident tiles (no cross-wave
// reduction), and handed on as MFMA operand images in LDS.  Apply products are shared out
// over the waves by tile; their epilogue runs in the layout the product comes out in, next to
// the tile rows fetched from LDS in that same layout, and ends in 128-bit stores.
//
// Both feature maps (the rows of Q and K are mapped while they are staged); ELU + 1 on the streaming
// kernels, which walk K, V twice, and here, fp16 d = 64, backward: 1024 slices x 197 rows 52.6 -> 44.2 us,
// 32 x 100 11.8 -> 7.5.
//
//   forward    stage K, V, Q | barrier | 4 waves: S | barrier | wave w: O rows of tile w
//   backward   see resident_bwd_kernel (dS is built while dQ is applied)
#include "cotten_launch.h"
#include "cotten_mfma_core.h"

namespace cotten {
namespace {

using namespace mfma;

constexpr int kWaves = 16;
constexpr int kThreads = 64 * kWaves;
constexpr int kMaxTiles = 13;                  // N <= 208
constexpr int kBlockBytes = 4 * kTileBytes;    // [khat | v | q(hat) | dO] tiles of 16 rows
constexpr int kKt = 0, kVt = kTileBytes, kQt = 2 * kTileBytes, kGt = 3 * kTileBytes;

template <class F>
struct Lds {
  static constexpr int kImages = kMaxTiles * kBlockBytes;          // three operand images
  static constexpr int kLive = kImages + 3 * F::kImageBytes;       // one int per tile
  static constexpr int kInv = kLive + 16 * 4;                      // 1/r per tile: 16 q rows, 16 k rows
  static constexpr int kDots = kInv + kMaxTiles * 2 * TR * 4;     // <S, dS> per state block
  static constexpr int kBytes = kDots + 4 * 4;
};

extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

struct Args {
  const unsigned char* Q;
  const unsigned char* K;
  const unsigned char* V;
  const unsigned char* dO;
  const uint8_t* mask;
  unsigned char* O;
  unsigned char* dQ;
  unsigned char* dK;
  unsigned char* dV;
  int H, N, slices;
  Strides st;
  float scale, eps;
  const float* scales;  // per-slice scale, or nullptr
  float* dlog;          // backward: <S, dS> per slice, or nullptr
  // S = sum_j m_j khat_j^T v_j of every slice as the caller keeps it from the forward to the
  // backward call ([slices][d][d] floats, row-major, without the scale), or nullptr
  float* saved;
  int d;                // head dimension (states are D x D, zero beyond d)
};

// The wave's tile: rows 16*tile + r8 + 8h.  `want` bit h: the row takes part.
template <bool USE_Y>
__device__ __forceinline__ void load_tile(Raw& r, const Lane& L, const Src& src, int tile,
                                          int want) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = tile * TR + L.r8 + 8 * h;
    const uint32_t off =
        src.offset(row, (want >> h) & 1, L);
    r.x[h] = __builtin_amdgcn_raw_buffer_load_b128(src.x, off, 0, 0);
    if (USE_Y) r.y[h] = __builtin_amdgcn_raw_buffer_load_b128(src.y, off, 0, 0);
    else r.y[h] = u32x4_t{0, 0, 0, 0};
  }
  r.live = want;
}

// Valid-key bits of the wave's tile in a slice (bit h: row 16*tile + r8 + 8h); all rows
// count when there is no mask, none when the slice does not exist.
__device__ __forceinline__ int key_rows(const Args& a, const Lane& L, int slice, int tile) {
  if (slice >= a.slices) return 0;
  if (a.mask == nullptr) return 3;
  const uint8_t* mask = a.mask + static_cast<size_t>(slice / a.H) * a.N;
  int keys = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = tile * TR + L.r8 + 8 * h;
    if (row < a.N) keys |= static_cast<int>(mask[row] != 0) << h;
  }
  return keys;
}

// Issues the loads of the wave's tile of `slice` (none, at no cost, if the slice or the tile
// does not exist): PARTS bit 0 = K and V, of which rows that are not valid keys are not read;
// bit 1 = Q (and dO).
template <bool BWD, int PARTS = 3>
__device__ __forceinline__ void fetch(Raw& rq, Raw& rk, const Args& a, const Lane& L, int slice,
                                      int tile, int keys) {
  const bool ok = slice < a.slices;
  const size_t base = ok ? a.st.slice_base(slice, a.H) : 0;
  int rows = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h)
    rows |= static_cast<int>(ok && tile * TR + L.r8 + 8 * h < a.N) << h;
  if (PARTS & 1) {
    const Src kv_src(a.K + base, a.V + base, a.N, a.st.row);
    load_tile<true>(rk, L, kv_src, tile, rows & keys);
  }
  if (PARTS & 2) {
    const Src q_src(a.Q + base, (BWD ? a.dO : a.Q) + base, a.N, a.st.row);
    load_tile<BWD>(rq, L, q_src, tile, rows);
  }
}

// 1/r of the 16 tile rows, from the load layout to where any wave can pick them up by row.
__device__ __forceinline__ void publish_inv(float* dst, const Lane& L, const float (&inv)[2]) {
  if (L.ch == 0) {
    dst[L.r8] = inv[0];
    dst[L.r8 + 8] = inv[1];
  }
}

// A block as it is (fp32, unscaled) into the caller's d x d array: the lane holds column
// c0 + lane%32 of rows r0 + 8j + 4*(lane/32) .. +3, so 32 lanes write 128 contiguous bytes.
template <class Acc>
__device__ __forceinline__ void save_block(const Acc& acc, const Lane& L, int r0, int c0, float* save_to, int d) {
  const int c = c0 + (L.lane & 31);
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = r0 + 8 * j + 4 * (L.lane >> 5) + v;
      if (r < d && c < d) save_to[r * d + c] = acc.v[4 * j + v];
    }
}

// One wave per state block: walks all kMaxTiles resident tiles and then writes its block into
// the images.  Tiles that contribute nothing must hold zeros.  The operands of the next
// kAhead tiles are requested from LDS before the matrix cores start on a tile (the scheduler
// is held to that order: left alone it funnels every tile through one register set, and each
// LDS read then waits for the product before it).
// Images are written with wide stores from an accumulator that holds the block the other way
// round: the natural image needs the transposed block, i.e. the operands swapped (a second
// accumulation, far cheaper than narrow image writes).
template <class F, bool NATURAL, bool TRANSPOSED>
__device__ __forceinline__ void build_state(const Lane& L, int block, int x_off, int y_off,
                                            float scale, unsigned char* natural,
                                            unsigned char* transposed,
                                            const unsigned char* other_natural = nullptr,
                                            float* dot_out = nullptr, float* save_to = nullptr,
                                            int d = 0) {
  typedef typename F::BlockAcc Acc;
  constexpr int kAhead = 3;
  static_assert(kAhead < kMaxTiles, "prefetch depth");
  Acc acc_t, acc_n;
  acc_t.zero();
  acc_n.zero();
  typename Acc::Frag ring[kAhead];
#pragma unroll
  for (int t = 0; t < kAhead; ++t)
    ring[t] = Acc::fetch(smem + t * kBlockBytes + x_off, smem + t * kBlockBytes + y_off, L, block);
#pragma unroll
  for (int t = 0; t < kMaxTiles; ++t) {
    const typename Acc::Frag f = ring[t % kAhead];
    __builtin_amdgcn_sched_barrier(0);
    if (t + kAhead < kMaxTiles) {
      const unsigned char* blk = smem + (t + kAhead) * kBlockBytes;
      ring[t % kAhead] = Acc::fetch(blk + x_off, blk + y_off, L, block);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (TRANSPOSED) acc_t.mma(f);
    if (NATURAL) acc_n.mma_swapped(f);
  }
  const int r0 = Acc::block_row0(block), c0 = Acc::block_col0(block);
  if (TRANSPOSED) acc_t.write_image(L, r0, c0, scale, transposed);
  if (NATURAL) acc_n.write_image(L, c0, r0, scale, natural);
  if (TRANSPOSED && save_to != nullptr) save_block(acc_t, L, r0, c0, save_to, d);
  // <this state, the state whose natural image is given>, this wave's block of it
  if (NATURAL && dot_out != nullptr) {
    const float dot = wave_sum(acc_n.dot_image(L, c0, r0, other_natural));
    if (L.lane == 0) *dot_out = dot;
  }
}

// Zero rows for the two tiles at Xt and Yt.
__device__ __forceinline__ void clear_tiles(const Lane& L, unsigned char* Xt, unsigned char* Yt) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int off = (L.r8 + 8 * h) * kTileStride + L.ch * 16;
    *reinterpret_cast<u32x4_t*>(Xt + off) = u32x4_t{0, 0, 0, 0};
    *reinterpret_cast<u32x4_t*>(Yt + off) = u32x4_t{0, 0, 0, 0};
  }
}

// Both kernels are persistent: a workgroup takes slices blockIdx.x, blockIdx.x + gridDim.x, ...
// and, as soon as one slice is staged in LDS, issues the loads of its next one, which then
// travel while the states are built and the products applied.

template <class F>
__global__ __launch_bounds__(kThreads) void resident_fwd_kernel(const Args a) {
  const Lane L0;
  const int N = a.N, tile = L0.wave, stride = gridDim.x;
  const int n_tiles = (N + TR - 1) / TR;
  unsigned char* blk = smem + tile * kBlockBytes;
  unsigned char* img = smem + Lds<F>::kImages;
  float* invs = reinterpret_cast<float*>(smem + Lds<F>::kInv) + tile * 2 * TR;
  const bool mine = tile < n_tiles;
  if (!mine && tile < kMaxTiles) {  // absent tiles stay zero for the whole kernel
    clear_tiles(L0, blk + kKt, blk + kVt);
    clear_tiles(L0, blk + kQt, blk + kGt);
  }

  int slice = blockIdx.x;
  Raw rq, rk;
  // The first slice: only K and V are requested at once (every compute unit asks at the same
  // moment, and the first phase needs nothing else); Q follows when those have arrived.
  fetch<false, 1>(rq, rk, a, L0, slice, tile, key_rows(a, L0, slice, tile));
  int keys = key_rows(a, L0, slice + stride, tile);
  // Per slice (B = workgroup barrier):
  //   1  tile waves stage K, V                                                       B
  //   2  waves 12-15 build S (at raised priority: everyone waits for it); tile waves
  //      stage Q and issue the loads of the next slice                               B
  //   3  wave w finishes the O rows of tile w (phase 1 of the next slice may start at once:
  //      it writes only the K, V tiles, which nobody reads any more)
  for (int iter = 0; slice < a.slices; slice += stride, ++iter) {
    {
      const Lane L = L0.again();
      if (mine) {
        float inv[2];
        if (__ballot(rk.live != 0) != 0)
          stage<F, mapped_mode<F>(), true>(rk, L, a.eps, blk + kKt, blk + kVt, inv, L.ch * 16 < a.st.row.bytes);
        else
          clear_tiles(L, blk + kKt, blk + kVt);
      }
      if (iter == 0) fetch<false, 2>(rq, rk, a, L, slice, tile, 0);
    }
    __syncthreads();
    {
      const Lane L = L0.again();
      constexpr int kB = F::BlockAcc::kBlocks;
      if (tile >= kWaves - kB) {  // O = qhat S: contraction over rows of S -> transposed image
        __builtin_amdgcn_s_setprio(3);
        const float scale = a.scales != nullptr ? a.scales[slice] : a.scale;
        build_state<F, false, true>(
            L, tile - (kWaves - kB), kKt, kVt, scale, nullptr, img, nullptr, nullptr,
            a.saved != nullptr ? a.saved + static_cast<size_t>(slice) * a.d * a.d : nullptr, a.d);
        __builtin_amdgcn_s_setprio(0);
      }
      if (mine) {
        float inv[2];
        // ELU + 1: phi(q) goes through the product, and 1/r is 1
        stage<F, F::kMap == kMapElu1 ? kXFeature : kXRaw, false>(rq, L, a.eps, blk + kQt, blk + kGt, inv,
                                                                 L.ch * 16 < a.st.row.bytes);
        publish_inv(invs, L, inv);
        fetch<false>(rq, rk, a, L, slice + stride, tile, keys);
        keys = key_rows(a, L, slice + 2 * stride, tile);
      }
    }
    __syncthreads();
    if (mine) {
      const Lane L = L0.again();
      typename F::TileRows xq;
      xq.load(blk + kQt, L);
      const float inv_r = invs[L.i16];
      typename F::Operand W;
      W.load(img, L);
      f32x4_t out[F::NT];
      F::apply(xq, W, out);
      float o[2 * F::EPL];
      product_rows<F>(out, o);
#pragma unroll
      for (int i = 0; i < 2 * F::EPL; ++i) o[i] *= inv_r;
      const int row = tile * TR + L.i16;
      if (row < N)
        store_product_row<F, kStoreStreamed>(a.O + a.st.slice_base(slice, a.H), row, a.st.row, L, o);
    }
  }
}

// One tile of an apply product, finished and stored:
//   kind 0  dQ = (g - qhat (qhat.g)) / r_q,  g = dO W      (W = scale * S, natural image)
//   kind 1  dV = khat W                                     (W = scale * dS, transposed image;
//                                                            khat is zero on masked rows)
//   kind 2  dK = (h - khat (khat.h)) / r_k,  h = v W       (W = scale * dS, natural image;
//                                                            1/r_k is zero on masked rows)
// (ELU + 1: phi(q), phi(k) in place of the unit rows, dQ = g phi'(q), dK = h phi'(k))
// Tiles without a valid key get zero rows of dK and dV without touching LDS.
template <class F>
__device__ __forceinline__ void apply_tile(const Lane& L, int kind, int t, int N,
                                           const typename F::Operand& W, const int* live,
                                           const float* invs, unsigned char* dst,
                                           RowAddr row_addr) {
  const unsigned char* tb = smem + t * kBlockBytes;
  const int row = t * TR + L.i16;
  float p[2 * F::EPL];
  if (kind != 0 && live[t] == 0) {
#pragma unroll
    for (int c = 0; c < 2 * F::EPL; ++c) p[c] = 0.0f;
  } else {
    typename F::TileRows x;
    x.load(tb + (kind == 0 ? kGt : kind == 1 ? kKt : kVt), L);
    f32x4_t out[F::NT];
    F::apply(x, W, out);
    product_rows<F>(out, p);
    if (kind != 1) {
      typename F::TileRows e;
      e.load(tb + (kind == 0 ? kQt : kKt), L);
      if (F::kMap == kMapElu1) feature_grad_rows<F>(p, e);
      else project_rows<F, true>(p, e, invs[t * 2 * TR + (kind == 0 ? 0 : TR) + L.i16], L);
    }
  }
  if (row < N) store_product_row<F, kStoreStreamed>(dst, row, row_addr, L, p);
}

// Backward, per slice (B = workgroup barrier):
//   1  tile waves stage Q, dO and request Q, dO of the next slice                    B
//   2  waves 12-15 build dS (one block each, at raised priority: everyone waits for it);
//      tile waves stage K, V and request K, V of the next slice                      B
//   3  waves 12-15 build S;  waves 0-11 apply dV and dK, which need only dS: waves 2i, 2i+1
//      take tiles i, i+6, i+12, one product each, so that every SIMD gets both kinds    B
//   4  wave w applies dQ of tile w                                                    B
template <class F>
__global__ __launch_bounds__(kThreads) void resident_bwd_kernel(const Args a) {
  const Lane L0;
  const int N = a.N, tile = L0.wave, stride = gridDim.x;
  const int n_tiles = (N + TR - 1) / TR;
  unsigned char* blk = smem + tile * kBlockBytes;
  unsigned char* img_s = smem + Lds<F>::kImages;              // scale * S, natural
  unsigned char* img_ds = img_s + F::kImageBytes;             // scale * dS, natural
  unsigned char* img_dst = img_ds + F::kImageBytes;           // scale * dS, transposed
  int* live = reinterpret_cast<int*>(smem + Lds<F>::kLive);
  float* invs = reinterpret_cast<float*>(smem + Lds<F>::kInv);
  const bool mine = tile < n_tiles;
  if (!mine && tile < kMaxTiles) {  // absent tiles stay zero for the whole kernel
    clear_tiles(L0, blk + kKt, blk + kVt);
    clear_tiles(L0, blk + kQt, blk + kGt);
  }
  constexpr int kB = F::BlockAcc::kBlocks, kApplyWaves = kWaves - kB;
  static_assert(kB == 4 && kWaves == 16 && kMaxTiles <= 16, "wave roles below");
  const int kv_kind = 1 + ((tile + (tile >> 2)) & 1);  // phase 3: dV or dK

  int slice = blockIdx.x;
  Raw rq, rk;
  // Loads are requested as early as the registers that receive them are free: everything of the
  // first slice at once, Q and dO of the next slice as soon as those of the current one are
  // staged, its K and V as soon as the current ones are (measured against requesting the next
  // slice in one go after phase 2, and K, V of the first slice only after Q, dO: 18.3 against
  // 21.0 us at 512 slices of 200 rows).
  const int first_keys = key_rows(a, L0, slice, tile);
  fetch<true>(rq, rk, a, L0, slice, tile, first_keys);
  int keys = key_rows(a, L0, slice + stride, tile);
  float* dots = reinterpret_cast<float*>(smem + Lds<F>::kDots);
  for (int iter = 0; slice < a.slices; slice += stride, ++iter) {
    const size_t base = a.st.slice_base(slice, a.H);
    const float scale = a.scales != nullptr ? a.scales[slice] : a.scale;
    {
      const Lane L = L0.again();
      if (mine) {
        float inv[2];
        stage<F, mapped_mode<F>(), true>(rq, L, a.eps, blk + kQt, blk + kGt, inv, L.ch * 16 < a.st.row.bytes);
        publish_inv(invs + tile * 2 * TR, L, inv);
      }
      // Q, dO of the next slice are requested as soon as their registers are free
      if (mine) fetch<true, 2>(rq, rk, a, L, slice + stride, tile, 0);
    }
    __syncthreads();
    {
      const Lane L = L0.again();
      if (tile >= kApplyWaves) {
        // dV = khat dS -> transposed image;  h = v dS^T -> natural image
        __builtin_amdgcn_s_setprio(3);  // the other waves wait for this at the next barrier
        build_state<F, true, true>(L, tile - kApplyWaves, kQt, kGt, scale, img_ds, img_dst);
        __builtin_amdgcn_s_setprio(0);
      }
      if (mine) {
        // A tile without a valid key adds nothing to S, and its dK, dV rows are plain zeros.
        const bool any_key = __ballot(rk.live != 0) != 0;
        if (any_key) {
          float inv[2];
          stage<F, mapped_mode<F>(), true>(rk, L, a.eps, blk + kKt, blk + kVt, inv, L.ch * 16 < a.st.row.bytes);
          publish_inv(invs + tile * 2 * TR + TR, L, inv);
        } else {
          clear_tiles(L, blk + kKt, blk + kVt);
        }
        if (L.lane == 0) live[tile] = any_key;
        fetch<true, 1>(rq, rk, a, L, slice + stride, tile, keys);
        keys = key_rows(a, L, slice + 2 * stride, tile);
      }
    }
    __syncthreads();
    if (tile >= kApplyWaves) {
      // g = dO S^T: contraction over columns of S -> natural image.  With dlog wanted: this
      // block of <sum_j khat_j^T v_j, scale * dS (its image)>
      const Lane L = L0.again();
      __builtin_amdgcn_s_setprio(3);
      build_state<F, true, false>(L, tile - kApplyWaves, kKt, kVt, scale, img_s, nullptr, img_ds,
                     a.dlog != nullptr ? dots + (tile - kApplyWaves) : nullptr);
      __builtin_amdgcn_s_setprio(0);
    } else {
      const Lane L = L0.again();
      typename F::Operand W;
      W.load(kv_kind == 1 ? img_dst : img_ds, L);
      unsigned char* dst = (kv_kind == 1 ? a.dV : a.dK) + base;
#pragma unroll 1
      for (int t = tile >> 1; t < n_tiles; t += kApplyWaves / 2)
        apply_tile<F>(L, kv_kind, t, N, W, live, invs, dst, a.st.row);
    }
    __syncthreads();
    // d loss / d log(scale) = sum_i dO_i . O_i = <S, scale * dS>, blocks in order
    if (a.dlog != nullptr && threadIdx.x == 0)
      a.dlog[slice] = ((dots[0] + dots[1]) + dots[2]) + dots[3];
    if (mine) {
      const Lane L = L0.again();
      typename F::Operand W;
      W.load(img_s, L);
      apply_tile<F>(L, 0, tile, N, W, live, invs, a.dQ + base, a.st.row);
    }
    __syncthreads();  // the tiles and images are rewritten for the next slice
  }
}

// ---- sequences of a few tiles: a workgroup of a wave per tile and slice, several on a compute unit ------
//
// Up to 128 rows.  The persistent kernels above hold a compute unit with sixteen waves whatever the length, and slices
// follow one another on it; here every slice has a workgroup of four or eight waves, 27 (forward) or 37 KB of LDS for four, and
// their phases overlap.  The states are built as above, a 32 x 32 block per wave (the same sums); own rows are
// held in the layout of the products by the time the operand images go over the tiles.
// Bound by the way to memory and back of a workgroup while few run, by memory beyond.  Forward / backward, us (left-padded lengths
// uniform in 0 ... N, over the same buffers), the persistent kernels and these, bf16 d = 64: 16 slices x 50 rows 4.4 / 6.3, 3.3 / 4.4;  512 x 50
// 6.2 / 10.1, 3.7 / 5.5;  4096 x 50 31.3 / 62.5, 15.8 / 28.8;  16 x 100 4.6 / 6.9, 3.8 / 5.4;  512 x 100 7.0 / 11.7, 4.9 / 7.7;  2048 x 128 21.5 / 41.5,
// 19.4 / 33.8;  d = 32, 2048 x 20 14.4 / 28.8, 5.6 / 11.6;  2048 x 128 19.4 / 37.5, 10.8 / 24.5.  Without a mask 512 x 100 6.3 / 11.5, 4.7 / 7.7; the
// forward of 2048 ... 6000 slices x 80 ... 128 rows of 128 bytes loses 1 ... 6 % where the buffers stay in the memory-side cache (2048 x 128 22.0,
// 23.0) and gains up to 5 % where they do not (4096 x 96 41.0, 39.5).  (K and V requested together with the mask, and what is masked
// dropped on arrival: as fast for 16 x 50, 6 % slower at 512 x 50, 2048 x 128 30 % and 20 %, where the masked rows cost traffic.)

// Valid-key bits of the wave's tile, see key_rows (no branch, the slice exists).
__device__ __forceinline__ int short_key_rows(const Args& a, const Lane& L, int bh, int tile) {
  int keys = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = tile * TR + L.r8 + 8 * h;
    const uint8_t key = a.mask == nullptr ? 1 : a.mask[static_cast<size_t>(bh / a.H) * a.N + (row < a.N ? row : 0)];
    keys |= static_cast<int>(row < a.N && key != 0) << h;
  }
  return keys;
}

// Forward.  DIRECT: rows of Q narrower than 128 bytes come straight in the layout of the products (d = 32, 2048 x 128
// 17.6 us through LDS, 14.9 this way; with rows of 128 bytes, 64 of which a load then takes, 512 x 50 4.7, 5.0).
template <class F, int WAVES, bool DIRECT>
__global__ __launch_bounds__(64 * WAVES, 4) void short_fwd_kernel(const Args a) {
  typedef typename F::BlockAcc Acc;
  constexpr int kStride = (DIRECT ? 2 : 3) * kTileBytes;  // of a tile: khat, v, q
  const Lane L;
  const int bh = blockIdx.x, tile = L.wave, N = a.N;
  const size_t base = a.st.slice_base(bh, a.H);
  const int row = tile * TR + L.i16;
  unsigned char* blk = smem + tile * kStride;
  float* invs = reinterpret_cast<float*>(smem + WAVES * kStride) + tile * TR;
  OwnRaw<1> own;
  {
    Raw rk, rq;
    const int keys = short_key_rows(a, L, bh, tile);
    if (DIRECT) load_own<1>(own, L, Buffers(a.Q + base, N, a.st.row), a.st.row, tile * TR, row < N);
    fetch<false, DIRECT ? 1 : 3>(rq, rk, a, L, bh, tile, keys);
    const bool cols = L.ch * 16 < a.st.row.bytes;
    float inv[2];
    stage<F, mapped_mode<F>(), true>(rk, L, a.eps, blk + kKt, blk + kVt, inv, cols);
    if (!DIRECT) {
      stage<F, F::kMap == kMapElu1 ? kXFeature : kXRaw, false>(rq, L, a.eps, blk + kQt, nullptr, inv, cols);
      publish_inv(invs, L, inv);
    }
  }
  __syncthreads();
  const bool builds = tile < Acc::kBlocks;
  const int r0 = Acc::block_row0(tile), c0 = Acc::block_col0(tile);
  Acc state;
  if (builds) {
    state.zero();
#pragma unroll
    for (int t = 0; t < WAVES; ++t) state.mma(Acc::fetch(smem + t * kStride + kKt, smem + t * kStride + kVt, L, tile));
  }
  // cosine map: the raw rows go through the product and 1/r is applied to the result; ELU + 1: phi(q), and 1
  typename F::TileRows x;
  float factor = 1.0f;
  if (!DIRECT) {
    x.load(blk + kQt, L);
    factor = invs[L.i16];
  } else {
    float f[2 * F::EPL];
    own_values<F, 1>(own, 0, f);
    if (F::kMap == kMapElu1) {
#pragma unroll
      for (int i = 0; i < 2 * F::EPL; ++i)
        f[i] = elu1_or_zero(f[i], (row < N) & (64 * (i / F::EPL) + 16 * L.g16 < a.st.row.bytes));
      x.set(f);
    } else {
      x.set(own.r[0][0], own.r[0][1]);
      float ss = 0.0f;
#pragma unroll
      for (int i = 0; i < 2 * F::EPL; ++i) ss += f[i] * f[i];
      factor = inv_norm_or_zero(row_sum_groups(ss, L), a.eps, row < N);
    }
  }
  __syncthreads();  // nobody reads the tiles any more
  if (builds) {
    state.write_image(L, r0, c0, a.scales != nullptr ? a.scales[bh] : a.scale, smem);
    if (a.saved != nullptr) save_block(state, L, r0, c0, a.saved + static_cast<size_t>(bh) * a.d * a.d, a.d);
  }
  __syncthreads();
  if (tile * TR >= N) return;
  typename F::Operand W;
  W.load(smem, L);
  f32x4_t out[F::NT];
  F::apply(x, W, out);
  float o[2 * F::EPL];
  product_rows<F>(out, o);
#pragma unroll
  for (int i = 0; i < 2 * F::EPL; ++i) o[i] *= factor;
  if (row < N) store_product_row<F, kStoreStreamed>(a.O + base, row, a.st.row, L, o);
}

template <class F, int WAVES>
struct ShortLds {
  static constexpr int kForwardDirect = WAVES * 2 * kTileBytes, kForward = WAVES * (3 * kTileBytes + TR * 4);
  static_assert(kForwardDirect >= F::kImageBytes, "the image goes over the tiles");
  static constexpr int kSpace = WAVES * kBlockBytes > 3 * F::kImageBytes ? WAVES * kBlockBytes : 3 * F::kImageBytes;
  static constexpr int kInv = kSpace, kDots = kInv + WAVES * 2 * TR * 4;
  static constexpr int kBackward = kDots + 4 * 4;
};

template <class F, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 4) void short_bwd_kernel(const Args a) {
  typedef typename F::BlockAcc Acc;
  typedef ShortLds<F, WAVES> Lds;
  constexpr int kB = Acc::kBlocks;
  static_assert(kB == 4 && (WAVES == 4 || WAVES == 8), "wave roles below");
  const Lane L;
  const int bh = blockIdx.x, tile = L.wave;
  const size_t base = a.st.slice_base(bh, a.H);
  unsigned char* blk = smem + tile * kBlockBytes;
  unsigned char *img_s = smem, *img_ds = img_s + F::kImageBytes, *img_dst = img_ds + F::kImageBytes;
  float* invs = reinterpret_cast<float*>(smem + Lds::kInv) + tile * 2 * TR;
  float* dots = reinterpret_cast<float*>(smem + Lds::kDots);
  const bool cols = L.ch * 16 < a.st.row.bytes;
  Raw rq, rk;
  fetch<true>(rq, rk, a, L, bh, tile, short_key_rows(a, L, bh, tile));
  float inv[2];
  stage<F, mapped_mode<F>(), true>(rk, L, a.eps, blk + kKt, blk + kVt, inv, cols);
  publish_inv(invs + TR, L, inv);
  stage<F, mapped_mode<F>(), true>(rq, L, a.eps, blk + kQt, blk + kGt, inv, cols);
  publish_inv(invs, L, inv);
  const bool any_key = __ballot(rk.live != 0) != 0;
  __syncthreads();
  // the wave's own rows, and a block of dS and of S (eight waves: of one of them)
  typename F::TileRows q, g, k, v;
  q.load(blk + kQt, L);
  g.load(blk + kGt, L);
  k.load(blk + kKt, L);
  v.load(blk + kVt, L);
  const float inv_q = invs[L.i16], inv_k = invs[TR + L.i16];
  const int block = tile % kB;
  const bool has_ds = WAVES == kB || tile < kB, has_s = WAVES == kB || tile >= kB;
  Acc ds_t, ds_n, s_n;
  ds_t.zero();
  ds_n.zero();
  s_n.zero();
  if (has_ds) {
#pragma unroll
    for (int t = 0; t < WAVES; ++t) {
      const typename Acc::Frag f = Acc::fetch(smem + t * kBlockBytes + kQt, smem + t * kBlockBytes + kGt, L, block);
      ds_t.mma(f);
      ds_n.mma_swapped(f);
    }
  }
  if (has_s) {
#pragma unroll
    for (int t = 0; t < WAVES; ++t)
      s_n.mma_swapped(Acc::fetch(smem + t * kBlockBytes + kKt, smem + t * kBlockBytes + kVt, L, block));
  }
  __syncthreads();  // the images go over the tiles
  const float scale = a.scales != nullptr ? a.scales[bh] : a.scale;
  const int r0 = Acc::block_row0(block), c0 = Acc::block_col0(block);
  if (has_ds) {
    ds_t.write_image(L, r0, c0, scale, img_dst);
    ds_n.write_image(L, c0, r0, scale, img_ds);
  }
  if (has_s) s_n.write_image(L, c0, r0, scale, img_s);
  __syncthreads();
  // d loss / d log(scale) = sum_i dO_i . O_i = <S, scale * dS>, blocks in order
  if (a.dlog != nullptr) {
    if (has_s) {
      const float dot = wave_sum(s_n.dot_image(L, c0, r0, img_ds));
      if (L.lane == 0) dots[block] = dot;
    }
    __syncthreads();
    if (threadIdx.x == 0) a.dlog[bh] = ((dots[0] + dots[1]) + dots[2]) + dots[3];
  }
  // (see apply_tile)
  const int row = tile * TR + L.i16;
  if (tile * TR >= a.N) return;
  const auto product = [&](const typename F::TileRows& x, const unsigned char* image, float (&p)[2 * F::EPL]) {
    typename F::Operand W;
    W.load(image, L);
    f32x4_t out[F::NT];
    F::apply(x, W, out);
    product_rows<F>(out, p);
  };
  const auto finish = [&](float (&p)[2 * F::EPL], typename F::TileRows& e, float inv_r) {
    if (F::kMap == kMapElu1) feature_grad_rows<F>(p, e);
    else project_rows<F, true>(p, e, inv_r, L);
  };
  float p[2 * F::EPL];
  product(g, img_s, p);
  finish(p, q, inv_q);
  if (row < a.N) store_product_row<F, kStoreStreamed>(a.dQ + base, row, a.st.row, L, p);
#pragma unroll
  for (int c = 0; c < 2 * F::EPL; ++c) p[c] = 0.0f;
  if (any_key) product(k, img_dst, p);
  if (row < a.N) store_product_row<F, kStoreStreamed>(a.dV + base, row, a.st.row, L, p);
  if (any_key) {
    product(v, img_ds, p);
    finish(p, k, inv_k);
  }
  if (row < a.N) store_product_row<F, kStoreStreamed>(a.dK + base, row, a.st.row, L, p);
}

// ---- causal variant on the matrix cores ------------------------------------------------------
// Row i attends the valid keys j <= i.  With the whole slice in LDS this is done tile pair by
// tile pair, (query tile t, key tile u <= t), all pairs independent:
//
//     P^T  = Khat_u Q_t^T          16 keys x 16 queries, two 16x16x32 MFMAs (contraction over d)
//     O_t^T += V_u^T P^T           16x16x16 MFMAs, one per 16 output columns
//
// A 16x16 MFMA result leaves lane (j, g) with rows 4g .. 4g+3 of column j - exactly the k a
// lane of a 16x16x16 B operand holds - so P (rounded to the element type, diagonal tile cut to
// its lower triangle) goes into the second product without moving between lanes; the A
// operand V_u^T comes from the transposing LDS read, with its columns picked so that the
// result lands in the product layout of the other kernels.  Wave t owns query tile t (and,
// in the backward, key tile t: t + 1 pairs in one role, n - t in the other, the same work for
// every wave).  Backward, with G^T = V_u dO_t^T on the same support:
//     dQhat_t^T += Khat_u^T G^T                         (as query tile t, over u <= t)
//     dV_u^T    += dO_t^T P,    H_u^T += Qhat_t^T G     (as key tile u, over t >= u)
// and the row-norm Jacobians as everywhere else.
// Served here: 16-bit rows of at most 208 positions (launch_causal() in cotten_causal.hip says when).

// A wave per tile: four, eight or thirteen.
template <int WAVES>
struct CausalLds {
  static constexpr int kLive = WAVES * kBlockBytes;  // one int per tile
  static constexpr int kInv = kLive + 16 * 4;        // 1/r per tile: 16 q rows, 16 k rows
  static constexpr int kBytes = kInv + WAVES * 2 * TR * 4;
};

template <class F, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 4) void causal_fwd_kernel(const Args a) {
  const Lane L0;
  const int N = a.N, tile = L0.wave, slice = blockIdx.x;
  const int n_tiles = (N + TR - 1) / TR;
  unsigned char* blk = smem + tile * kBlockBytes;
  int* live = reinterpret_cast<int*>(smem + CausalLds<WAVES>::kLive);
  float* invs = reinterpret_cast<float*>(smem + CausalLds<WAVES>::kInv) + tile * 2 * TR;
  const bool mine = tile < n_tiles;
  Raw rq, rk;
  const int from = mine ? slice : a.slices;  // a slice that does not exist: nothing is loaded
  fetch<false>(rq, rk, a, L0, from, tile, key_rows(a, L0, from, tile));
  if (mine) {
    float inv[2];
    const bool any_key = __ballot(rk.live != 0) != 0;
    if (any_key) stage<F, kXNormalized, true>(rk, L0, a.eps, blk + kKt, blk + kVt, inv);
    if (L0.lane == 0) live[tile] = any_key;
    stage<F, kXRaw, false>(rq, L0, a.eps, blk + kQt, blk + kGt, inv);
    publish_inv(invs, L0, inv);
  }
  __syncthreads();
  if (!mine) return;
  const Lane L = L0.again();
  typename F::TileRows xq;
  xq.load(blk + kQt, L);
  f32x4_t out[F::NT];
#pragma unroll
  for (int nt = 0; nt < F::NT; ++nt) out[nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int u = 0; u <= tile; ++u) {
    if (live[u] == 0) continue;  // no valid key in the tile (uniform)
    const unsigned char* ub = smem + u * kBlockBytes;
    typename F::TileRows xk;
    xk.load(ub + kKt, L);
    f32x4_t pt = F::dots(xk, xq);  // [key 4g+v][query i16]
    if (u == tile) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (4 * L.g16 + v > L.i16) pt[v] = 0.0f;
    }
    F::add_transposed_product(ub + kVt, L, F::weights(pt), out);
  }
  float o[2 * F::EPL];
  product_rows<F>(out, o);
  const float factor = invs[L.i16] * (a.scales != nullptr ? a.scales[slice] : a.scale);
#pragma unroll
  for (int i = 0; i < 2 * F::EPL; ++i) o[i] *= factor;
  const int row = tile * TR + L.i16;
  if (row < N)
    store_product_row<F, kStoreStreamed>(a.O + a.st.slice_base(slice, a.H), row, a.st.row, L, o);
}

// RAW: dQ, dK and dV from the wave's own rows as they are, as the walk over chunks has them, and not from rows rounded after
// their division by r (bf16, 300 slices x 50 rows, distance of dV from 64 bits 2.9e-3, otherwise 3.3e-3).
template <class F, int WAVES, bool RAW>
__global__ __launch_bounds__(64 * WAVES, 4) void causal_bwd_kernel(const Args a) {
  const Lane L0;
  const int N = a.N, tile = L0.wave, slice = blockIdx.x;
  const int n_tiles = (N + TR - 1) / TR;
  unsigned char* blk = smem + tile * kBlockBytes;
  int* live = reinterpret_cast<int*>(smem + CausalLds<WAVES>::kLive);
  float* invs = reinterpret_cast<float*>(smem + CausalLds<WAVES>::kInv) + tile * 2 * TR;
  const bool mine = tile < n_tiles;
  Raw rq, rk;
  const int from = mine ? slice : a.slices;  // a slice that does not exist: nothing is loaded
  fetch<true>(rq, rk, a, L0, from, tile, key_rows(a, L0, from, tile));
  OwnRaw<1> own_queries, own_keys;
  if (RAW) {
    const int row = tile * TR + L0.i16;
    const size_t at = static_cast<size_t>(slice / a.H) * N + (row < N ? row : 0), base = a.st.slice_base(slice, a.H);
    const bool key = row < N && (a.mask == nullptr || a.mask[at] != 0);
    load_own<1>(own_queries, L0, Buffers(a.Q + base, N, a.st.row), a.st.row, tile * TR, row < N);
    load_own<1>(own_keys, L0, Buffers(a.K + base, N, a.st.row), a.st.row, tile * TR, key);
  }
  if (mine) {
    float inv[2];
    stage<F, kXNormalized, true>(rq, L0, a.eps, blk + kQt, blk + kGt, inv);
    publish_inv(invs, L0, inv);
    const bool any_key = __ballot(rk.live != 0) != 0;
    if (any_key) {
      stage<F, kXNormalized, true, true>(rk, L0, a.eps, blk + kKt, blk + kVt, inv);
      publish_inv(invs + TR, L0, inv);
    }
    if (L0.lane == 0) live[tile] = any_key;
  }
  __syncthreads();
  if (!mine) return;
  const Lane L = L0.again();
  const size_t base = a.st.slice_base(slice, a.H);
  const float scale = a.scales != nullptr ? a.scales[slice] : a.scale;
  const int row = tile * TR + L.i16;

  {  // as query tile: dQ
    typename F::TileRows xg;
    xg.load(blk + kGt, L);
    f32x4_t acc[F::NT];
#pragma unroll
    for (int nt = 0; nt < F::NT; ++nt) acc[nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int u = 0; u <= tile; ++u) {
      if (live[u] == 0) continue;
      const unsigned char* ub = smem + u * kBlockBytes;
      typename F::TileRows xv;
      xv.load(ub + kVt, L);
      f32x4_t gt = F::dots(xv, xg);  // [key 4g+v][query i16] = v_key . dO_query
      if (u == tile) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (4 * L.g16 + v > L.i16) gt[v] = 0.0f;
      }
      F::add_transposed_product(ub + kKt, L, F::weights(gt), acc);
    }
    float g[2 * F::EPL];
    product_rows<F>(acc, g);
#pragma unroll
    for (int i = 0; i < 2 * F::EPL; ++i) g[i] *= scale;
    typename F::TileRows e;
    if (RAW) {
      e.set(own_queries.r[0][0], own_queries.r[0][1]);
      project_rows_raw<F>(g, e, invs[L.i16], L);
    } else {
      e.load(blk + kQt, L);
      project_rows<F, false>(g, e, invs[L.i16], L);
    }
    if (row < N) store_product_row<F, kStoreStreamed>(a.dQ + base, row, a.st.row, L, g);
  }

  {  // as key tile: dK, dV
    float dk[2 * F::EPL], dv[2 * F::EPL];
    if (live[tile] == 0) {
#pragma unroll
      for (int i = 0; i < 2 * F::EPL; ++i) dk[i] = dv[i] = 0.0f;
    } else {
      typename F::TileRows xk, xv;
      const float inv_k = invs[TR + L.i16];
      if (RAW) xk.set(own_keys.r[0][0], own_keys.r[0][1]);
      else xk.load(blk + kKt, L);
      xv.load(blk + kVt, L);
      f32x4_t av[F::NT], ah[F::NT];
#pragma unroll
      for (int nt = 0; nt < F::NT; ++nt) av[nt] = ah[nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      for (int t = tile; t < n_tiles; ++t) {
        const unsigned char* tb = smem + t * kBlockBytes;
        typename F::TileRows xq, xg;
        xq.load(tb + kQt, L);
        xg.load(tb + kGt, L);
        f32x4_t p = F::dots(xq, xk);   // [query 4g+v][key i16] = qhat_query . khat_key
        if (RAW) p *= inv_k;
        f32x4_t gg = F::dots(xg, xv);  // [query 4g+v][key i16] = dO_query . v_key
        if (t == tile) {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (L.i16 > 4 * L.g16 + v) p[v] = gg[v] = 0.0f;
        }
        F::add_transposed_product(tb + kGt, L, F::weights(p), av);
        F::add_transposed_product(tb + kQt, L, F::weights(gg), ah);
      }
      product_rows<F>(av, dv);
      product_rows<F>(ah, dk);
#pragma unroll
      for (int i = 0; i < 2 * F::EPL; ++i) {
        dv[i] *= scale;
        dk[i] *= scale;
      }
      if (RAW) project_rows_raw<F>(dk, xk, inv_k, L);
      else project_rows<F, false>(dk, xk, inv_k, L);
      zero_masked(inv_k, dk, dv);
    }
    if (row < N) {
      store_product_row<F, kStoreStreamed>(a.dK + base, row, a.st.row, L, dk);
      store_product_row<F, kStoreStreamed>(a.dV + base, row, a.st.row, L, dv);
    }
  }
}

// Persistent workgroups: one per compute unit of the current device (the LDS admits no second
// one), 256 on MI355X.  Asked once per device.
int compute_units() {
  constexpr int kMaxDevices = 64;
  static int cached[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

Args make_args(const Problem& p) {
  Args a{};
  a.Q = static_cast<const unsigned char*>(p.Q);
  a.K = static_cast<const unsigned char*>(p.K);
  a.V = static_cast<const unsigned char*>(p.V);
  a.dO = static_cast<const unsigned char*>(p.dO);
  a.mask = p.mask;
  a.O = static_cast<unsigned char*>(p.O);
  a.dQ = static_cast<unsigned char*>(p.dQ);
  a.dK = static_cast<unsigned char*>(p.dK);
  a.dV = static_cast<unsigned char*>(p.dV);
  a.H = p.H;
  a.N = p.N;
  a.slices = p.B * p.H;
  a.st = Strides{p.stride_batch * p.elem_bytes(), p.stride_head * p.elem_bytes(),
                 RowAddr{static_cast<int>(p.stride_row * p.elem_bytes()),
                         static_cast<int>(p.D * p.elem_bytes())}};
  a.scale = p.scale;
  a.eps = p.eps;
  a.scales = p.slice_scale;
  a.dlog = p.dlog_scale;
  a.saved = p.saved_state;
  a.d = p.D;
  return a;
}

template <class F, int WAVES>
hipError_t run_short(const Problem& p, const Args& a, bool bwd) {
  const auto launch = [&](auto kernel, int bytes) {
    const hipError_t err = grant_dynamic_lds(reinterpret_cast<const void*>(kernel), bytes);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(a.slices)), dim3(64 * WAVES), bytes, p.stream, a);
    return hipGetLastError();
  };
  if (bwd) return launch(short_bwd_kernel<F, WAVES>, ShortLds<F, WAVES>::kBackward);
  return a.st.row.bytes < kRowBytes ? launch(short_fwd_kernel<F, WAVES, true>, ShortLds<F, WAVES>::kForwardDirect)
                                    : launch(short_fwd_kernel<F, WAVES, false>, ShortLds<F, WAVES>::kForward);
}

template <class F>
hipError_t run(const Problem& p, bool bwd) {
  const Args a = make_args(p);
  // (A launch has fewer than 2^32 threads: with more slices than that admits, 2^24 of up to 64 rows or 2^23 of up to 128, the persistent
  // kernels below, whose launches have as many workgroups as there are compute units.)
  const int short_waves = p.N <= 4 * TR ? 4 : 8;
  if (p.N <= 8 * TR && static_cast<int64_t>(a.slices) * 64 * short_waves < int64_t{1} << 32)
    return short_waves == 4 ? run_short<F, 4>(p, a, bwd) : run_short<F, 8>(p, a, bwd);
  const int units = compute_units();
  const dim3 grid(static_cast<unsigned>(a.slices < units ? a.slices : units));
  const size_t lds = Lds<F>::kBytes;
  // The backward never reads a kept state here: with the slice in LDS K and V are fetched once
  // whether S is rebuilt or not, and reading d x d floats per slice would only add traffic (at
  // d = 64 and 200 rows the state is 16 KB next to 25 KB per tensor: measured 23.1 against
  // 18.4 us at 512 slices).
  const void* kern = bwd ? reinterpret_cast<const void*>(resident_bwd_kernel<F>)
                         : reinterpret_cast<const void*>(resident_fwd_kernel<F>);
  const hipError_t err = grant_dynamic_lds(kern, static_cast<int>(lds));
  if (err != hipSuccess) return err;
  if (bwd)
    hipLaunchKernelGGL(resident_bwd_kernel<F>, grid, dim3(kThreads), lds, p.stream, a);
  else
    hipLaunchKernelGGL(resident_fwd_kernel<F>, grid, dim3(kThreads), lds, p.stream, a);
  return hipGetLastError();
}

}  // namespace

template <class F, int WAVES>
hipError_t run_causal(const Problem& p, bool bwd) {
  const Args a = make_args(p);
  const auto launch = [&](auto kernel) {
    constexpr int lds = CausalLds<WAVES>::kBytes;
    const hipError_t err = grant_dynamic_lds(reinterpret_cast<const void*>(kernel), lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(a.slices)), dim3(64 * WAVES), lds, p.stream, a);
    return hipGetLastError();
  };
  // (RAW from 257 slices on: dV is then as far from 64 bits as the walk over chunks leaves it, bf16, 300 x 50 2.88e-3, without 3.33e-3.  Fewer slices
  // wait for its loads of the own rows: 16 and 128 slices x 50 rows 4.6 and 4.8 us, RAW 4.8 and 5.0.)
  if constexpr (WAVES == 4) {
    if (bwd && a.slices > 256) return launch(causal_bwd_kernel<F, WAVES, true>);
  }
  return bwd ? launch(causal_bwd_kernel<F, WAVES, false>) : launch(causal_fwd_kernel<F, WAVES>);
}
template <class F>
hipError_t run_causal(const Problem& p, bool bwd) {
  return p.N <= 4 * TR ? run_causal<F, 4>(p, bwd) : p.N <= 8 * TR ? run_causal<F, 8>(p, bwd) : run_causal<F, kMaxTiles>(p, bwd);
}

bool resident_supports(int dtype, int D, int N) {
  return (dtype == 1 || dtype == 2) && (D == 64 || D == 32 || D == 16) && N <= kMaxTiles * mfma::TR;
}

static_assert(kCausalChunkRows == kMaxTiles * mfma::TR, "what the LDS holds is one chunk");

bool causal_resident_supports(int dtype, int D) {
  return dtype == 0 ? (D == 32 || D == 16) : (D == 64 || D == 32 || D == 16);
}

hipError_t launch_resident_causal(const Problem& p, bool bwd) {
  if (!resident_supports(p.dtype, p.D, p.N)) return hipErrorInvalidValue;
  return p.dtype == 1 ? run_causal<Bf16x64>(p, bwd) : run_causal<F16x64>(p, bwd);
}

namespace {
hipError_t run_mapped(const Problem& p, bool bwd) {
  if (p.feature_map == kMapElu1)
    return p.dtype == 1 ? run<WithElu1<Bf16x64>>(p, bwd) : run<WithElu1<F16x64>>(p, bwd);
  return p.dtype == 1 ? run<Bf16x64>(p, bwd) : run<F16x64>(p, bwd);
}
}  // namespace

hipError_t launch_resident_fwd(const Problem& p) { return run_mapped(p, false); }

hipError_t launch_resident_bwd(const Problem& p) { return run_mapped(p, true); }

}  // namespace cotten
