// Causal variant of the cosine attention (row i attends the valid keys j <= i), the form the
// paper's bidirectional model leaves out ("no causal mask"):
//
//     S_i = sum_{j <= i} m_j khat_j^T v_j          O_i = scale * qhat_i S_i
//
// as a walk over chunks of 16 * WAVES rows by one workgroup, one 16-row tile per wave, with the
// d x d state of everything before the chunk carried along:
//
//     O_c = scale * ( Qhat_c S_before  +  tril(Qhat_c Khat_c^T) V_c ),     S_before += Khat_c^T V_c
//
// and, for the backward, one walk forwards (dQ needs the prefix state) and one walk backwards
// (dK, dV need the suffix state T = sum_{i later} qhat_i^T dO_i), as two roles of one launch:
//
//     G = dO_c V_c^T, P = Qhat_c Khat_c^T          (lower triangle, valid keys)
//     g_c  = scale * (dO_c S_before^T + G Khat_c)           -> dQ
//     dV_c = scale * (Khat_c T_after + P^T dO_c)
//     h_c  = scale * (V_c T_after^T  + G^T Qhat_c)          -> dK
//
// Everything is a matrix-core product: the triangle tile pair by tile pair (`dots`,
// `add_transposed_product` of the element format), the carried state as operand images in LDS
// (`apply`), its update one 32 x 32 block per wave.  What a wave needs of its own rows it loads
// straight in the layout of the products; only the rows that other waves read go through LDS.
//
// Measured (fwd / bwd, us): fp32 d = 64, 128 slices x 200 rows 13.4 / 30.6, where a scan on the vector
// units (16 rows per step) took 89 / 149; bf16 d = 64, 256 x 1001 rows 28 / 67, where 208-row
// chunks joined by states in memory took 56 / 101 (three launches, 13 * 14 / 2 tile pairs per chunk
// instead of 8 * 9 / 2 per 128 rows).  Bound: bf16 - the forward by memory, at about 4 TB/s with two chunks of loads in
// flight per wave (with one, and the bytes of the key mask waited for before the loads of their rows, 33.2; 64 x 1001
// rows 20.3, now 17.1), the backward by waits, with one: 249 MB, what its two roles share read twice, at 3.7 TB/s (without
// any product the same loads and stores take 54 of its 67 us; two chunks in flight: it has no registers for more); fp32 - latency:
// with its products as bf16 pieces (44.5 -> 43.5 per step) the matrix rate no longer is (mask bytes ahead: 32 x 2048
// rows, d = 64, forward 79 -> 71.6;  1024 x 200 backward 149 -> 144;  8 x 200 backward 12.7, now 13.2).
//
// 16-bit results differ from those of 208-row chunks in the places where sums are rounded, by about as much
// as either differs from a 64-bit evaluation (bf16, 256 x 1001 rows: 3e-3; from 64 bits 2.9e-3 ... 3.3e-3
// there, 2.5e-3 here: the state in two images, dV from raw keys).
#include "cotten_launch.h"
#include "cotten_mfma_core.h"

namespace cotten {
namespace {

using namespace mfma;

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
  int H, N;
  int segments, segment_chunks;  // a slice is cut into segments of so many chunks, a workgroup each
  Strides st;
  float scale, eps;
  const float* scales;
  // sums of the states before / after every segment, [slice][segment][D*D] floats row-major, or
  // nullptr: the workgroup walks the chunks before (after) its segment for their states alone
  const float* before;
  const float* after;
};

enum Role { kO = 0, kDq = 1, kDkDv = 2, kDv = 3, kDk = 4 };
constexpr bool role_up(int role) { return role == kO || role == kDq; }  // ascending chunks
// Rows of two pieces: one image set per workgroup is what lets two of them share a compute unit, so
// dV and dK, which need different sets, are roles of their own there.
template <int P>
constexpr bool separate_dv_dk() { return P == 2; }

// An element of the carried state is a sum over all the rows before (after), and what a row gets from it
// may be a small difference of such elements.  With 16-bit rows the state therefore has two operand
// images, the second of what the first leaves off: 16 (bf16) and 22 bits, where the tile pairs
// keep sums of 32 bits.  Keys and values with a common component that the queries do not see, bf16,
// distance of O from a 64-bit evaluation, one image and two: N = 200 2.1e-2 and 4.5e-3 (tile pairs alone
// 4.7e-3); N = 1001 6.3e-2 and 4.3e-3 (ordinary inputs 2.9e-3 and 2.5e-3).  Forward / backward, us, one and
// two: bf16 256 slices x 1001 rows 31.7 / 75.2, 32.6 / 76.7; 64 x 1001 19.5 / 27.4, 19.9 / 28.3.
template <class F>
constexpr int state_images() { return F::kElemBytes == 2 ? 2 : 1; }

// LDS: [per wave: x tile, y tile, P pieces each][one flag per wave][size of each state block][one
// (forward) or two sets of P x P operand images, each state_images() times]
template <class F, int P, int WAVES>
struct ScanLds {
  static constexpr int kWaveBytes = 2 * P * F::kTileBytes;
  static constexpr int kLive = WAVES * kWaveBytes;
  static constexpr int kSizes = kLive + 8 * 4;
  static constexpr int kImages = kLive + 16 * 4;
  static constexpr int kSet = state_images<F>() * P * P * F::kImageBytes;
  // `carried`: there is more than one chunk
  static constexpr int bytes(bool bwd, bool carried) {
    return kImages + (carried ? (bwd && !separate_dv_dk<P>() ? 2 : 1) * kSet : 0);
  }
};

// A 16-row tile of a tensor pair on its way to LDS (load layout): piece [h][c] is bytes 128 c + 16 ch
// .. + 15 of row r8 + 8 h; `live` bit h: the row takes part.
template <int P>
struct SharedRaw {
  u32x4_t x[2][P], y[2][P];
  int live;
};

// The key mask of a sequence; without one every row of it takes part.  Its bytes are requested a chunk before the rows that
// they decide on, and tested when those are requested: a wait for them would be one for every load before them.
struct Keys {
  __amdgpu_buffer_rsrc_t r;
  int N;
  bool all;
  __device__ __forceinline__ Keys(const uint8_t* mask, int n)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(mask), 0, mask == nullptr ? 0 : n, 0x00020000)),
        N(n), all(mask == nullptr) {}
  // (rows outside the sequence lie outside the buffer: zero, no traffic)
  __device__ __forceinline__ unsigned request(int row) const {
    return __builtin_amdgcn_raw_buffer_load_b8(r, row, 0, 0);
  }
  __device__ __forceinline__ bool test(unsigned byte, int row) const { return all ? row < N : byte != 0; }
};

template <int P>
__device__ __forceinline__ void load_shared(SharedRaw<P>& t, const Lane& L, const Buffers& X, const Buffers& Y,
                                            RowAddr addr, int row0, int bits) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const bool live = ((bits >> h) & 1) != 0;
    // rows narrower than 128 bytes (one piece only): the lanes beyond them load zeros
    const uint32_t off = (live && L.ch * 16 < addr.bytes)
                             ? static_cast<uint32_t>(row0 + L.r8 + 8 * h) * addr.stride + L.ch * 16
                             : kOutOfBuffer;
#pragma unroll
    for (int c = 0; c < P; ++c) {
      t.x[h][c] = __builtin_amdgcn_raw_buffer_load_b128(X.r, off + c * kRowBytes, 0, 0);
      t.y[h][c] = __builtin_amdgcn_raw_buffer_load_b128(Y.r, off + c * kRowBytes, 0, 0);
    }
  }
  t.live = bits;
}

// The shared tile into LDS: xhat pieces, then y pieces.
template <class F, int P>
__device__ __forceinline__ void stage_shared(const SharedRaw<P>& t, const Lane& L, float eps,
                                             unsigned char* tiles) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float f[P][F::EPL];
    float ss = 0.0f;
#pragma unroll
    for (int c = 0; c < P; ++c) {
      F::unpack(t.x[h][c], f[c]);
#pragma unroll
      for (int i = 0; i < F::EPL; ++i) ss += f[c][i] * f[c][i];
    }
    const float inv = inv_norm_or_zero(row_sum8(ss), eps, ((t.live >> h) & 1) != 0);
#pragma unroll
    for (int c = 0; c < P; ++c) {
#pragma unroll
      for (int i = 0; i < F::EPL; ++i) f[c][i] *= inv;
      F::put(tiles + c * F::kTileBytes, L.r8 + 8 * h, L.ch, f[c]);
      if (!F::kPieces) F::put_raw(tiles + (P + c) * F::kTileBytes, L.r8 + 8 * h, L.ch, t.y[h][c]);
    }
  }
  if (!F::kPieces) return;
  float top = 0.0f;
#pragma unroll
  for (int c = 0; c < P; ++c) top = F::largest_raw(t.y[0][c], F::largest_raw(t.y[1][c], top));
  write_pieces<F>(top, [&](auto inf) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < P; ++c)
        F::template put_raw<decltype(inf)::value>(tiles + (P + c) * F::kTileBytes, L.r8 + 8 * h, L.ch, t.y[h][c]);
  });
}

// States of any size in half operand images: an image holds 2^-e of the state and what comes out of a product
// with it is multiplied by 2^e.  e = 0 while the state stays below 2^15 in magnitude (the usual
// case: nothing is rounded differently then), otherwise what brings its largest value there.
constexpr float kHalfTop = 32768.0f;
struct HalfRange {
  float factor, back;  // uniform, in scalar registers
  __device__ __forceinline__ explicit HalfRange(float largest) {
    const int exponent = (__builtin_amdgcn_readfirstlane(__float_as_int(largest)) >> 23) & 0xff;
    const int e = exponent > 141 && exponent < 255 ? exponent - 141 : 0;  // 2^15 = 0.5 * 2^16, biased 142
    factor = __int_as_float((127 - e) << 23);
    back = __int_as_float((127 + e) << 23);
  }
};

// What a wave carries of the state: one 32 x 32 block.  NATURAL / TRANSPOSED: which operand images
// it keeps up to date.  The transposed one is written four values at a time from an accumulator that
// holds the block as it is, the natural one likewise from one that holds it transposed (operands
// swapped).  Where both are kept there is one accumulator (registers; matrix-core time) and the
// natural image is written by pairs of columns: write_across().
template <class F, int P, bool NATURAL, bool TRANSPOSED>
struct Carried {
  typedef typename F::BlockAcc Acc;
  static constexpr int kPerPair = Acc::kBlocks, kBlocks = P * P * kPerPair;
  static constexpr bool kScatter = NATURAL && TRANSPOSED;
  static constexpr bool kPlain = TRANSPOSED || kScatter, kSwapped = NATURAL && !kScatter;
  Acc plain, swapped;
  int p, q, block;  // block `block` of piece p of x against piece q of y
  __device__ __forceinline__ explicit Carried(int index)
      : p(index / kPerPair / P), q(index / kPerPair % P), block(index % kPerPair) {
    if (kPlain) plain.zero();
    if (kSwapped) swapped.zero();
  }
  // M: a row-major state of side D
  __device__ __forceinline__ void read(const float* __restrict__ M, int D, const Lane& L) {
    const int r0 = p * F::D + Acc::block_row0(block), c0 = q * F::D + Acc::block_col0(block);
    const int col = Acc::run_col(L);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int run = Acc::run_row(j, L);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (kPlain) plain.v[4 * j + i] = M[(r0 + run + i) * D + c0 + col];
        if (kSwapped) swapped.v[4 * j + i] = M[(r0 + col) * D + c0 + run + i];
      }
    }
  }
  __device__ __forceinline__ void add(const unsigned char* tiles, const Lane& L) {
    const typename Acc::Frag f =
        Acc::fetch(tiles + p * F::kTileBytes, tiles + (P + q) * F::kTileBytes, L, block);
    if (kPlain) plain.mma(f);
    if (kSwapped) swapped.mma_swapped(f);
  }
  // The largest magnitude of the block, as far as it matters: 0 if it is below kHalfTop.
  __device__ __forceinline__ float size() const {
    const Acc& acc = kPlain ? plain : swapped;
    float top = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) top = fmaxf(top, fabsf(acc.v[i]));
    if (__builtin_amdgcn_ballot_w64(top >= kHalfTop) == 0) return 0.0f;
#pragma unroll
    for (int w = 1; w < 64; w <<= 1) top = fmaxf(top, __shfl_xor(top, w));
    return top;
  }
  // the images of factor * state
  __device__ __forceinline__ void write(unsigned char* natural, unsigned char* transposed, float factor,
                                        const Lane& L) const {
    const int r0 = Acc::block_row0(block), c0 = Acc::block_col0(block);
    Acc straight = plain, turned = swapped;  // (those that are not kept are not looked at)
#pragma unroll
    for (int k = 0; k < state_images<F>(); ++k) {
      const int at = (k * P * P + p * P + q) * F::kImageBytes;
      const float f = k == 0 ? factor : 1.0f;
      if (k > 0) {
        if (kPlain) left_over(straight, factor);
        if (kSwapped) left_over(turned, factor);
      }
      if (TRANSPOSED) straight.write_image(L, r0, c0, f, transposed + at);
      if (kSwapped) turned.write_image(L, c0, r0, f, natural + at);
      if (kScatter) write_across(straight, f, natural + at, r0, c0, L);
    }
  }
  // The natural image from an accumulator that holds the block as it is: pairs of columns, the second from the
  // neighbouring lane (even lanes write the first two rows of a run, odd lanes the last two).
  static __device__ __forceinline__ void write_across(const Acc& acc, float factor, unsigned char* image, int r0, int c0,
                                                      const Lane& L) {
    const bool odd = (L.lane & 1) != 0;
    Lane zero = L;
    zero.set(0);
    unsigned char* at = image + F::image_offset(r0 + Acc::run_row(0, L) + (odd ? 2 : 0), c0 + (Acc::run_col(L) & ~1));
    float top = 0.0f;
    if (F::kPieces) {
#pragma unroll
      for (int i = 0; i < 16; ++i) top = fmaxf(top, fabsf(acc.v[i]));
    }
    write_pieces<F>(top, [&](auto inf) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float first = acc.v[4 * j + i] * factor, second = acc.v[4 * j + 2 + i] * factor;
          const float mine = odd ? second : first;
          int sent = __builtin_bit_cast(int, odd ? first : second);  // (see quadrant_image)
          asm volatile("" : "+v"(sent));
          int got = __builtin_amdgcn_update_dpp(0, sent, 0xB1, 0xF, 0xF, true);  // lane ^ 1
          asm volatile("" : "+v"(got));
          const float other = __builtin_bit_cast(float, got);
          F::template write_pair_at<decltype(inf)::value>(at + F::image_offset(Acc::run_row(j, zero) + i, 0),
                                                          odd ? other : mine, odd ? mine : other);
        }
    });
  }
  // what the image of factor * state leaves off
  static __device__ __forceinline__ void left_over(Acc& acc, float factor) {
    if constexpr (state_images<F>() > 1) {
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        float v0 = acc.v[i] * factor, v1 = acc.v[i + 1] * factor;
        F::left_over(v0, v1);
        acc.v[i] = v0;
        acc.v[i + 1] = v1;
      }
    }
  }
};

// out[piece] = back * sum_c X[piece c] W(first + c * step) over the images of a set
template <class F, int P>
__device__ __forceinline__ void apply_set(const typename F::TileRows (&X)[P], const unsigned char* images,
                                          int first, int step, float back, const Lane& L, f32x4_t (&out)[F::NT]) {
  if constexpr (state_images<F>() == 1) {
#pragma unroll
    for (int c = 0; c < P; ++c) {
      typename F::Operand W;
      W.load(images + (first + c * step) * F::kImageBytes, L);
      if (c == 0) F::apply(X[c], W, out);
      else F::apply_onto(X[c], W, out);
    }
  } else {
    static_assert(P == 1, "16-bit rows are one piece");
#pragma unroll
    for (int nt = 0; nt < F::NT; ++nt) {
      out[nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < state_images<F>(); ++k)
        out[nt] = F::apply_columns(X[0], images + k * F::kImageBytes, nt, L, out[nt]);
    }
  }
  if (!F::kFloatRange) {
#pragma unroll
    for (int nt = 0; nt < F::NT; ++nt) out[nt] *= back;
  }
}

// 1/r of the lane's own row (0 if the row does not take part)
template <class F, int P>
__device__ __forceinline__ float own_inv(const typename F::TileRows (&x)[P], float eps, bool live, const Lane& L) {
  float ss = 0.0f;
#pragma unroll
  for (int c = 0; c < P; ++c) {
    float f[2 * F::EPL];
    x[c].unpack(f);
#pragma unroll
    for (int i = 0; i < 2 * F::EPL; ++i) ss += f[i] * f[i];
  }
  return inv_norm_or_zero(row_sum_groups(ss, L), eps, live);
}

// g <- (g - u (u.g)) / r over all pieces, from the raw rows x = r u:  (g - x (x.g) / r^2) / r
template <class F, int P>
__device__ __forceinline__ void project_own(float (&g)[P][2 * F::EPL], const typename F::TileRows (&x)[P],
                                            float inv_r, const Lane& L) {
  float proj = 0.0f;
#pragma unroll
  for (int c = 0; c < P; ++c) {
    float f[2 * F::EPL];
    x[c].unpack(f);
#pragma unroll
    for (int i = 0; i < 2 * F::EPL; ++i) proj += f[i] * g[c][i];
  }
  // one factor at a time: 1/r^2 alone leaves the fp32 range for rows next to zero, and (x.g) / r^3 for long ones
  proj = row_sum_groups(proj, L) * inv_r * inv_r;
#pragma unroll
  for (int c = 0; c < P; ++c) {
    float f[2 * F::EPL];
    x[c].unpack(f);
#pragma unroll
    for (int i = 0; i < 2 * F::EPL; ++i) g[c][i] = (g[c][i] - f[i] * proj) * inv_r;
  }
}

template <class F, int P>
__device__ __forceinline__ void store_own(unsigned char* dst, int row, int N, RowAddr addr, const Lane& L,
                                          const float (&o)[P][2 * F::EPL]) {
  if (row >= N) return;
#pragma unroll
  for (int c = 0; c < P; ++c)
    store_product_row<F, kStoreStreamed>(dst + c * kRowBytes, row,
                                         RowAddr{addr.stride, addr.bytes - c * kRowBytes}, L, o[c]);
}

// Per chunk (B = workgroup barrier):
//   stage the wave's shared tile (roles O, dQ: khat, v; role dK, dV: qhat, dO), write the state
//   carried so far into the operand images, request everything of the next chunk         B
//   own rows: carried state, then the tile pairs; epilogue, stores.  Then the waves with the
//   fewest pairs add the chunk to the carried state, one 32 x 32 block each              B
// UNMASKED: the kernel is for calls without a mask: nothing is requested for one, and one chunk of rows is on its way.
template <class F, int P, int WAVES, int ROLE, bool UNMASKED>
__device__ __forceinline__ void scan_segment(const Args& a, int bh, int segment) {
  typedef ScanLds<F, P, WAVES> Lds;
  typedef typename F::TileRows TileRows;
  constexpr bool kUp = role_up(ROLE), kTwoOwn = ROLE != kO && ROLE != kDv;
  constexpr int kState = F::D * P;
  const Lane L0;
  const Lane& L = L0;
  const int N = a.N, wave = L.wave;
  const int n_tiles = (N + TR - 1) / TR, chunks = (n_tiles + WAVES - 1) / WAVES;
  const size_t base = a.st.slice_base(bh, a.H);
  const RowAddr addr = a.st.row;
  const uint8_t* keys = UNMASKED || a.mask == nullptr ? nullptr : a.mask + static_cast<size_t>(bh / a.H) * N;
  const Keys shared_keys(kUp ? keys : nullptr, N), own_keys(kUp ? nullptr : keys, N);
  const float scale = a.scales != nullptr ? a.scales[bh] : a.scale;
  const Buffers sx((kUp ? a.K : a.Q) + base, N, addr), sy((kUp ? a.V : a.dO) + base, N, addr);
  const Buffers ox((kUp ? a.Q : a.K) + base, N, addr), oy((ROLE == kDq ? a.dO : a.V) + base, N, addr);

  const int first = segment * a.segment_chunks;
  const int last = first + a.segment_chunks < chunks ? first + a.segment_chunks : chunks;
  const float* given = kUp ? a.before : a.after;
  // the walk starts at the segment when the states around it are given, at the sequence's end otherwise
  const int begin = kUp ? (given != nullptr ? first : 0) : (given != nullptr ? last - 1 : chunks - 1);
  int steps = kUp ? last - begin : begin - first + 1;

  unsigned char* mine = smem + wave * Lds::kWaveBytes;
  unsigned char* natural = smem + Lds::kImages;
  unsigned char* transposed = smem + Lds::kImages + (ROLE == kDkDv ? Lds::kSet : 0);
  int* live = reinterpret_cast<int*>(smem + Lds::kLive);
  float* sizes = reinterpret_cast<float*>(smem + Lds::kSizes);

  // the state blocks go to the waves with the fewest tile pairs
  typedef Carried<F, P, ROLE != kO && ROLE != kDv, ROLE != kDq && ROLE != kDk> State;
  const int duty = kUp ? wave : WAVES - 1 - wave;
  const bool on_duty = duty < State::kBlocks;
  State state(on_duty ? duty : 0);
  const auto publish_size = [&] {
    static_assert(F::kFloatRange || (State::kBlocks <= 8 && WAVES <= 8), "place for the sizes");
    if (F::kFloatRange || !on_duty) return;
    const float top = state.size();
    if (L.lane == 0) sizes[duty] = top;
  };
  bool have = false;  // the images stand for something (uniform)
  if (given != nullptr && (kUp ? segment > 0 : segment < a.segments - 1)) {
    have = true;
    if (on_duty)
      state.read(given + (static_cast<size_t>(bh) * a.segments + segment) * kState * kState, kState, L);
    publish_size();
    if (!F::kFloatRange) __syncthreads();
  }

  const auto tile_of = [&](int step) { return (kUp ? begin + step : begin - step) * WAVES + wave; };
  const auto applies = [&](int step) { return kUp ? begin + step >= first : begin - step < last; };
  // (the backward of fp32 rows of one piece is at the registers of four waves per SIMD: its keys are read where they
  // are needed, 512 slices x 128 rows 18.2 us against 21.0, and where there is a mask: 512 x 400 rows 56.4, through an empty buffer 57.4)
  constexpr bool kKeysAhead = !UNMASKED && (ROLE == kO || F::kElemBytes == 2 || P == 2);
  struct KeyBytes {
    unsigned of[2];
  };
  const auto request_keys = [&](int step) {
    const int row0 = tile_of(step) * TR;
    KeyBytes b = {{0u, 0u}};
    if (kUp) {
      b.of[0] = shared_keys.request(row0 + L.r8);
      b.of[1] = shared_keys.request(row0 + L.r8 + 8);
    } else {
      b.of[0] = own_keys.request(row0 + L.i16);
    }
    return b;
  };
  // the rows of a chunk on their way
  struct Ahead {
    SharedRaw<P> shared;
    OwnRaw<P> nx, ny;
    bool live;
  };
  const auto request = [&](Ahead& t, int step, const KeyBytes& b, const Lane& L) {
    const int row0 = tile_of(step) * TR, row = row0 + L.r8;
    int bits = 0;
    if (!kUp) {
      bits = static_cast<int>(row < N) | static_cast<int>(row + 8 < N) << 1;
    } else if (kKeysAhead) {
      bits = static_cast<int>(shared_keys.test(b.of[0], row)) | static_cast<int>(shared_keys.test(b.of[1], row + 8)) << 1;
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (row + 8 * h < N) bits |= static_cast<int>(keys == nullptr || keys[row + 8 * h] != 0) << h;
    }
    load_shared<P>(t.shared, L, sx, sy, addr, row0, bits);
    if (applies(step)) {
      const int own = row0 + L.i16;
      if (kUp) t.live = own < N;
      else if (kKeysAhead) t.live = own_keys.test(b.of[0], own);
      else t.live = own < N && (keys == nullptr || keys[own] != 0);
      load_own<P>(t.nx, L, ox, addr, row0, t.live);
      if (kTwoOwn) load_own<P>(t.ny, L, oy, addr, row0, t.live);
    }
  };
  // The forward of 16-bit rows, which has the registers for it, keeps two chunks on their way where the mask decides on the rows, the others
  // one.  The second is requested when the first has come: both at once would come together (bf16 d = 64, 256 x 1001 rows, padded: one 33.2 us, two
  // at once 31.8, this 30.3).  Workgroups of four waves, which walk one chunk or two, keep one (bf16, 1024 x 50: two 6.3, one 6.0).
  constexpr int kAhead = !UNMASKED && ROLE == kO && F::kElemBytes == 2 && WAVES == 8 ? 2 : 1;
  Ahead ahead[kAhead];
  KeyBytes next_keys = {{0u, 0u}}, second_keys;
  {
    KeyBytes b[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) b[i] = kKeysAhead ? request_keys(i) : KeyBytes{{0u, 0u}};
    // (without the condition the fp32 forward of two pieces is compiled into one that waits more: 346 x 28 rows 6.1 us, 6.7; the others gain)
    if (kKeysAhead && (P == 1 || ROLE != kO || steps > kAhead)) next_keys = request_keys(kAhead);
    second_keys = b[kAhead - 1];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      ahead[i].live = false;
      if (i == 0) request(ahead[i], i, b[i], L);
    }
  }
  if (!kUp && keys != nullptr && steps > 4) {
    // Chunks below the first valid key of the segment get zeros and are not walked.  (Looking for it
    // costs a trip to memory before the walk: 16-bit, 256 x 1001 rows, left-padded, 93 -> 77 us;
    // with four chunks or fewer it is not worth it.)
    int lo = N;
#pragma unroll 4
    for (int row = first * WAVES * TR + static_cast<int>(threadIdx.x); row < last * WAVES * TR; row += 64 * WAVES)
      if (row < N && keys[row] != 0 && row < lo) lo = row;
#pragma unroll
    for (int w = 1; w < 64; w <<= 1) {
      const int other = __shfl_xor(lo, w);
      lo = other < lo ? other : lo;
    }
    if (L.lane == 0) live[wave] = lo;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) lo = live[w] < lo ? live[w] : lo;
    lo = __builtin_amdgcn_readfirstlane(lo);
    __syncthreads();
    steps = lo < N ? begin - lo / (WAVES * TR) + 1 : 0;
    const int below = lo < N ? lo / (WAVES * TR) : last;  // chunks first .. below-1
    float zeros[P][2 * F::EPL];
#pragma unroll
    for (int c = 0; c < P; ++c)
#pragma unroll
      for (int i = 0; i < 2 * F::EPL; ++i) zeros[c][i] = 0.0f;
#pragma unroll 1
    for (int t = first * WAVES + wave; t < below * WAVES; t += WAVES) {
      if (ROLE != kDk) store_own<F, P>(a.dV + base, t * TR + L.i16, N, addr, L, zeros);
      if (ROLE != kDv) store_own<F, P>(a.dK + base, t * TR + L.i16, N, addr, L, zeros);
    }
  }
  const auto walk = [&](int step, Ahead& now) {
    const Lane L = P == 1 ? L0.again() : L0;  // (registers: see Lane::again)
    SharedRaw<P>& shared = now.shared;
    const bool tile_live = __builtin_amdgcn_ballot_w64(shared.live != 0) != 0;
    if (tile_live) stage_shared<F, P>(shared, L, a.eps, mine);
    if (L.lane == 0) live[wave] = tile_live;
    float largest = 0.0f;  // of the state
    if (!F::kFloatRange && have) {
#pragma unroll
      for (int b = 0; b < State::kBlocks; ++b) largest = fmaxf(largest, sizes[b]);
    }
    const HalfRange range(largest);
    if (have && on_duty && applies(step)) state.write(natural, transposed, range.factor, L);
    TileRows x[P], y[P];
    own_rows<F, P, false>(now.nx, x);
    if (kTwoOwn) own_rows<F, P, true>(now.ny, y);
    const bool row_live = now.live;
    const int tile = tile_of(step);
    const KeyBytes bytes = next_keys;
    if (kKeysAhead) next_keys = request_keys(step + kAhead + 1);  // (a branch here would wait: 64 x 4096 rows backward 98 -> 105)
    if (kAhead == 2 && step == 0 && steps > 1) request(ahead[kAhead - 1], 1, second_keys, L);
    if (step + kAhead < steps) request(now, step + kAhead, bytes, L);
    __syncthreads();
    int flags = 0;  // bit u: tile u of the chunk has rows that take part
#pragma unroll
    for (int u = 0; u < WAVES; ++u) flags |= (live[u] != 0) << u;
    flags = __builtin_amdgcn_readfirstlane(flags);

    if (applies(step) && tile < n_tiles) {
      const int row = tile * TR + L.i16;
      if (kUp) {
        const TileRows(&own)[P] = ROLE == kO ? x : y;
        f32x4_t out[P][F::NT];
#pragma unroll
        for (int c = 0; c < P; ++c) {
          if (have) {
            if (ROLE == kO) apply_set<F, P>(own, transposed, c, P, range.back, L, out[c]);
            else apply_set<F, P>(own, natural, P * c, 1, range.back, L, out[c]);
          } else {
#pragma unroll
            for (int nt = 0; nt < F::NT; ++nt) out[c][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          }
        }
        // (No `unroll 1`: the compiler gives the wave's own tile, the last one, a copy of the body and spares the others its selects and
        // branches.  With it, forward / backward, us, bf16: 256 slices x 1001 rows 28.9 / 72.9, without 27.7 / 67.4;  32 x 300 8.0 / 15.1,
        // 7.6 / 13.3;  64 x 2000 30.5 / 51.7, 29.8 / 48.5.  The next tile's rows read ahead by hand: 27.6 / 68.9, fp32 spills.)
        for (int u = 0; u <= wave; ++u) {
          if (((flags >> u) & 1) == 0) continue;  // no valid key in the tile
          const unsigned char* tu = smem + u * Lds::kWaveBytes;
          // [key 4g+v][query i16]: khat . q (role O), v . dO (role dQ)
          f32x4_t pt = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int c = 0; c < P; ++c) {
            TileRows key;
            key.load(tu + ((ROLE == kO ? 0 : P) + c) * F::kTileBytes, L);
            pt = F::dots(key, own[c], pt);
          }
          if (u == wave) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (4 * L.g16 + v > L.i16) pt[v] = 0.0f;
          }
          // (khat . q is infinite in rows only that 1/r makes NaN anyway)
          const typename F::Weights w = F::template weights<ROLE != kO>(pt);
#pragma unroll
          for (int c = 0; c < P; ++c)
            F::add_transposed_product(tu + ((ROLE == kO ? P : 0) + c) * F::kTileBytes, L, w, out[c]);
        }
        const float inv_r = own_inv<F, P>(x, a.eps, row_live, L);
        const float factor = ROLE == kO ? inv_r * scale : scale;
        float o[P][2 * F::EPL];
#pragma unroll
        for (int c = 0; c < P; ++c) {
          product_rows<F>(out[c], o[c]);
#pragma unroll
          for (int i = 0; i < 2 * F::EPL; ++i) o[c][i] *= factor;
        }
        if (ROLE == kDq) project_own<F, P>(o, x, inv_r, L);
        store_own<F, P>((ROLE == kO ? a.O : a.dQ) + base, row, N, addr, L, o);
      } else {
        // dV, then dK: each product pair reads what the other does not, so doing them one after the
        // other costs no LDS reads and halves the accumulators in flight
        const bool any_key = __builtin_amdgcn_ballot_w64(row_live) != 0;
        const float inv_r = any_key ? own_inv<F, P>(x, a.eps, row_live, L) : 0.0f;
#pragma unroll
        for (int kind = 0; kind < 2; ++kind) {
          if (ROLE == (kind == 0 ? kDk : kDv)) continue;
          const Lane L = P == 1 ? L0.again() : L0;  // (registers: see Lane::again)
          float o[P][2 * F::EPL];
#pragma unroll
          for (int c = 0; c < P; ++c)
#pragma unroll
            for (int i = 0; i < 2 * F::EPL; ++i) o[c][i] = 0.0f;
          if (any_key) {
            const TileRows(&own)[P] = kind == 0 ? x : y;
            // tiles whose rows meet the own ones in dots(), and those the result is made of
            const int left = (kind == 0 ? 0 : P) * F::kTileBytes, right = (kind == 0 ? P : 0) * F::kTileBytes;
            f32x4_t out[P][F::NT];
#pragma unroll
            for (int c = 0; c < P; ++c) {
              if (have) {
                if (kind == 0) {
                  apply_set<F, P>(own, transposed, c, P, F::kFloatRange ? 1.0f : range.back * inv_r, L, out[c]);
                } else {
                  apply_set<F, P>(own, natural, P * c, 1, range.back, L, out[c]);
                }
              } else {
#pragma unroll
                for (int nt = 0; nt < F::NT; ++nt) out[c][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
              }
            }
            for (int t = wave; t < WAVES; ++t) {
              if (((flags >> t) & 1) == 0) continue;  // beyond the sequence
              const unsigned char* tt = smem + t * Lds::kWaveBytes;
              // [query 4g+v][key i16]: qhat . k (dV), dO . v (dK)
              f32x4_t p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int c = 0; c < P; ++c) {
                TileRows query;
                query.load(tt + left + c * F::kTileBytes, L);
                p = F::dots(query, own[c], p);
              }
              if (kind == 0 && !F::kFloatRange) p *= inv_r;  // qhat . khat fits a half, qhat . k may not
              if (t == wave) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                  if (L.i16 > 4 * L.g16 + v) p[v] = 0.0f;
              }
              const typename F::Weights w = kind == 0 ? F::weights(p) : F::template weights<true>(p);
#pragma unroll
              for (int c = 0; c < P; ++c) F::add_transposed_product(tt + right + c * F::kTileBytes, L, w, out[c]);
            }
            const float factor = kind == 0 && F::kFloatRange ? inv_r * scale : scale;
#pragma unroll
            for (int c = 0; c < P; ++c) {
              product_rows<F>(out[c], o[c]);
#pragma unroll
              for (int i = 0; i < 2 * F::EPL; ++i) o[c][i] *= factor;
            }
            if (kind == 1) project_own<F, P>(o, x, inv_r, L);
#pragma unroll
            for (int c = 0; c < P; ++c)
#pragma unroll
              for (int i = 0; i < 2 * F::EPL; ++i) o[c][i] = row_live ? o[c][i] : 0.0f;  // masked: exact zeros
          }
          store_own<F, P>((kind == 0 ? a.dV : a.dK) + base, row, N, addr, L, o);
        }
      }
    }
    if (step + 1 < steps && flags != 0) {
      const Lane L = P == 1 ? L0.again() : L0;  // (registers: see Lane::again)
      have = true;
      if (on_duty) {
#pragma unroll 2
        for (int u = 0; u < WAVES; ++u)
          if ((flags >> u) & 1) state.add(smem + u * Lds::kWaveBytes, L);
        publish_size();
      }
    }
    __syncthreads();  // the tiles and images are written again next
  };
#pragma unroll 1
  for (int step = 0; step < steps; step += kAhead) {
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      if (i == 0 || step + i < steps) walk(step + i, ahead[i]);
  }
}

template <class F, int P, int WAVES, bool UNMASKED>
__global__ __launch_bounds__(64 * WAVES, P == 1 ? 4 : 2) void causal_scan_fwd_kernel(const Args a) {
  scan_segment<F, P, WAVES, kO, UNMASKED>(a, blockIdx.x / a.segments, blockIdx.x % a.segments);
}

// blockIdx.y == 0: dQ.   blockIdx.y == 1: dK and dV, or (1, 2) dV, dK.
template <class F, int P, int WAVES, bool UNMASKED>
__global__ __launch_bounds__(64 * WAVES, P == 1 ? 4 : 2) void causal_scan_bwd_kernel(const Args a) {
  const int bh = blockIdx.x / a.segments, segment = blockIdx.x % a.segments;
  if (blockIdx.y == 0) scan_segment<F, P, WAVES, kDq, UNMASKED>(a, bh, segment);
  else if constexpr (!separate_dv_dk<P>()) scan_segment<F, P, WAVES, kDkDv, UNMASKED>(a, bh, segment);
  else if (blockIdx.y == 1) scan_segment<F, P, WAVES, kDv, UNMASKED>(a, bh, segment);
  else scan_segment<F, P, WAVES, kDk, UNMASKED>(a, bh, segment);
}

constexpr int kThreads = 256;

// Chunked matrix-core path: the states of the chunks, [slice][chunk][dd] floats, become in
// place the sums a chunk needs.  Block row 0: every S_c is replaced by the sum of the S before
// chunk c, added in chunk order; block row 1 (backward): every T_c, stored behind all the S,
// by the sum of the T after chunk c, added from the last chunk down.  One thread per four
// consecutive floats of a state; the values of up to kAhead chunks are requested together.
// The last S and the first T were never written and are not read.
__global__ __launch_bounds__(kThreads) void chunk_scan_kernel(float* states, int slices, int chunks,
                                                              int quads) {
  constexpr int kAhead = 8;
  const int id = blockIdx.x * kThreads + threadIdx.x;
  if (id >= slices * quads) return;
  const bool downwards = blockIdx.y == 1;
  f32x4_t* base = reinterpret_cast<f32x4_t*>(states) +
                  (static_cast<size_t>(blockIdx.y) * slices + id / quads) * chunks * quads + id % quads;
  f32x4_t run = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < chunks; s0 += kAhead) {
    f32x4_t own[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int step = s0 + j;  // chunk `step` counted from the end the sum starts at
      own[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if (step < chunks - 1)
        own[j] = base[static_cast<size_t>(downwards ? chunks - 1 - step : step) * quads];
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int step = s0 + j;
      if (step < chunks) {
        base[static_cast<size_t>(downwards ? chunks - 1 - step : step) * quads] = run;
        run += own[j];
      }
    }
  }
}


template <class F, int P, int WAVES>
hipError_t run_scan(const Problem& p, bool bwd) {
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
  a.st = Strides{p.stride_batch * p.elem_bytes(), p.stride_head * p.elem_bytes(),
                 RowAddr{static_cast<int>(p.stride_row * p.elem_bytes()),
                         static_cast<int>(p.D * p.elem_bytes())}};
  a.scale = p.scale;
  a.eps = p.eps;
  a.scales = p.slice_scale;
  const int slices = p.B * p.H, chunk_rows = 16 * WAVES, chunks = (p.N + chunk_rows - 1) / chunk_rows;
  a.segments = 1;
  a.segment_chunks = chunks;
  // Segments: about one workgroup per compute unit and role (16-bit rows, fp32 rows of 256 bytes), two
  // where the tiles are small and the matrix cores slow (fp32 rows of 128 bytes).  Measured with 1,
  // 2, 4, 8 segments (fwd / bwd, us):  bf16 d = 64, 256 slices x 1001 rows 32 / 77, 35 / 77, 45 / 91,
  // 68 / 120; 64 x 1001 29 / 53, 22 / 34, 19 / 29, 20 / 34;  fp32 d = 64, 128 x 200 22 / 35,
  // 16 / 30, 16 / 32; 32 x 2048 184 / 324, 128 / 192, 99 / 125, 83 / 107;  fp32 d = 32,
  // 128 x 1000 47 / 77, 41 / 63, 46 / 58.
  const int target = (P == 1 && F::kElemBytes == 4) ? 512 : 256;
  const int most = P == 1 && causal_chunks(p.N) > 1 ? causal_chunks(p.N) : 16;
  int n = (target + slices - 1) / slices;
  if (n > chunks) n = chunks;
  if (n > most) n = most;
  // The states around the segments: every workgroup walks the chunks before (after) its segment
  // itself, for their states alone, while that is little; from more than four segments on, and in a
  // forward with long segments or slow matrix cores, two launches ahead sum them up in the
  // workspace (where there is one: it holds causal_chunks(N) states per slice, none for one chunk).
  // 64 x 4096 bf16, 4 segments: 67 / 100 us walked, 52 / 106 us given; 8 segments: 69 / 127, 50 / 111.
  bool states_given = P == 1 && n > 1 && causal_chunks(p.N) > 1 &&
                      (n > 4 || (!bwd && (F::kElemBytes == 4 || p.N > 2048)));
  if (states_given) {
    constexpr int kMostRows = 16384;  // the key flags of a segment must fit LDS
    const int at_least = (p.N + kMostRows - 1) / kMostRows;
    if (n < at_least) n = at_least;
  }
  a.segment_chunks = (chunks + n - 1) / n;
  a.segments = (chunks + a.segment_chunks - 1) / a.segment_chunks;
  if (states_given) {
    if (p.workspace == nullptr || a.segments > causal_chunks(p.N)) return hipErrorInvalidValue;
    const int side = mfma_state_dim(p.dtype);
    hipError_t err = launch_chunk_states(p, a.segment_chunks * WAVES, a.segments, bwd);
    if (err != hipSuccess) return err;
    err = launch_chunk_scan(p.workspace, slices, a.segments, side * side, bwd, p.stream);
    if (err != hipSuccess) return err;
    a.before = p.workspace;
    a.after = p.workspace + static_cast<size_t>(slices) * a.segments * side * side;
  }
  const int lds = ScanLds<F, P, WAVES>::bytes(bwd, chunks > 1);
  const dim3 grid(static_cast<unsigned>(slices) * a.segments, bwd ? (separate_dv_dk<P>() ? 3 : 2) : 1);
  const auto launch = [&](auto kernel) {
    const hipError_t err =
        grant_dynamic_lds(reinterpret_cast<const void*>(kernel), ScanLds<F, P, WAVES>::bytes(bwd, true));
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kernel, grid, dim3(64 * WAVES), lds, p.stream, a);
    return hipGetLastError();
  };
  // Calls without a mask have kernels of their own where that gains (bytes of an empty buffer, us, and none): bf16 d = 64, forward 256 x 600 22.7,
  // 21.5; 128 x 318 10.3, 9.4; backward 21.7, 20.6; 256 x 1001 79.4, 80.5;  fp32 d = 64, backward 8 x 200 13.3, 12.9; 128 x 200 31.9, 31.5.  Not the
  // fp32 forward (8 x 2800 87.8, 91.6) nor fp32 d = 32 (backward 64 x 820 37.9, 43.7).
  // (16-bit rows in chunks of four tiles: forward only, see launch_causal)
  if (bwd) {
    if constexpr (F::kElemBytes == 2 && WAVES == 4) return hipErrorInvalidValue;
    else {
      if constexpr (F::kElemBytes == 2 || P == 2)
        if (p.mask == nullptr) return launch(causal_scan_bwd_kernel<F, P, WAVES, true>);
      return launch(causal_scan_bwd_kernel<F, P, WAVES, false>);
    }
  }
  if constexpr (F::kElemBytes == 2)
    if (p.mask == nullptr) return launch(causal_scan_fwd_kernel<F, P, WAVES, true>);
  return launch(causal_scan_fwd_kernel<F, P, WAVES, false>);
}

}  // namespace

hipError_t launch_chunk_scan(float* states, int slices, int chunks, int dd, bool with_queries,
                             hipStream_t stream) {
  const int quads = dd / 4;
  const dim3 grid((static_cast<unsigned>(slices) * quads + kThreads - 1) / kThreads,
                  with_queries ? 2 : 1);
  hipLaunchKernelGGL(chunk_scan_kernel, grid, dim3(kThreads), 0, stream, states, slices, chunks, quads);
  return hipGetLastError();
}

bool causal_supports(int D) { return D == 16 || D == 32 || D == 64; }

size_t causal_workspace_floats(int B, int H, int N, int D, int dtype, bool is_bwd) {
  const int chunks = causal_chunks(N);
  if (chunks < 2 || !causal_resident_supports(dtype, D)) return 0;
  const size_t side = static_cast<size_t>(mfma_state_dim(dtype));
  return static_cast<size_t>(B) * H * chunks * side * side * (is_bwd ? 2 : 1);
}

hipError_t launch_causal(const Problem& p, bool bwd) {
  if (!causal_resident_supports(p.dtype, p.D)) {
    if (p.dtype != 0 || p.D != 64) return hipErrorInvalidValue;
    return run_scan<F32x32, 2, 4>(p, bwd);
  }
  // fp32, a slice of at most 208 rows held in LDS whole (with fp32 products) and the walk, forward / backward, us,
  // d = 32:  8 slices x 200 rows 9.7 / 19.8, 7.7 / 9.8;  256 x 200 12.5 / 26.6, 11.8 / 20.5;  2048 x 200
  // 70 / 149, 42 / 113;  64 x 50 4.1 / 6.1, 4.1 / 6.1;  512 x 50 8.7 / 12.7, 5.6 / 10.3;  512 x 128 13.9 / 26.3,
  // 10.6 / 20.8
  if (p.dtype == 0) return run_scan<F32x32, 1, 4>(p, bwd);
  // 16-bit rows.  The walk reads what its two backward roles share twice; a slice of at most 208
  // rows held in LDS is read once: workgroups of four waves up to 64 rows (four on a compute unit), of eight up to 128 (two), of thirteen
  // beyond (one).  The backward always gains by it, the forward while the workgroups do not queue up.  us, walk and in LDS, bf16 d = 64,
  // with a key mask (left-padded lengths uniform in 0 ... N) and without, over the same buffers:
  //   forward   512 slices x 50 rows 3.9, 3.8 and 4.0, 3.7;  1024 x 50 5.0, 4.6 and 4.7, 4.4;  512 x 100 5.7, 5.0 and 5.3, 5.0;  1022 x 100 11.1, 9.0 and
  //             10.6, 10.4;  over fresh ones 2048 x 50 10.6, 11.0;  2048 x 100 20.2, 20.4;  256 x 200 9.5, 8.2;  512 x 200 11.6, 13.9
  //   backward  512 x 50 7.3, 5.8 and 6.9, 5.6;  4096 x 50 39.0, 27.2 and 42.5, 30.4;  (with sixteen waves whatever the length, 512 x 100 11.0,
  //             now 8.1;  2048 x 100 42.9, 28.8);  over fresh ones 512 x 200 29.1, 26.9
  // (1024 slices or more of 65 ... 128 rows, forward: chunks of 64 rows, whose carried state keeps more bits than the scores do: 2.65e-3 from
  // 64 bits at 1024 x 100, in LDS 2.88e-3.)
  const long slices = static_cast<long>(p.B) * p.H;
  const bool resident = causal_chunks(p.N) == 1 &&
                        (bwd || (p.N <= 64 ? slices <= 1024 : p.N <= 128 ? slices < 1024 : slices <= 256));
  if (resident) return launch_resident_causal(p, bwd);
  if (p.N <= 64 || (p.N <= 128 && slices >= 1024))
    return p.dtype == 1 ? run_scan<Bf16x64, 1, 4>(p, bwd) : run_scan<F16x64, 1, 4>(p, bwd);
  return p.dtype == 1 ? run_scan<Bf16x64, 1, 8>(p, bwd) : run_scan<F16x64, 1, 8>(p, bwd);
}

}  // namespace cotten
