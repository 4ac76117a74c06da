// Wide rows, sequences that are not cut: one workgroup per slice, every wave the owner of 32 columns of the results
// (fp32 d_h = 128 in both directions, 16-bit d_h = 128 in the backward).
//
//     S = sum_j xhat_j^T y_j       each wave one or two 32 x 32 blocks of it, over all rows
//     T = X W                      each wave 32 columns of T, its part of W held in registers
//
// The rows are walked in rounds: the waves stage a round in LDS together (mapped and cut into the operand
// format once for the whole workgroup), and every product of the round is taken from there.  The state
// goes from the accumulators through LDS, as the fp32 matrix that it is, into the registers of the waves
// that multiply by it, in either orientation.
//
//   forward    (K, V) -> S;   Q -> O = scale qhat S
//   backward   (K, V) -> S;   (Q, dO) -> dS and, in the same rounds, dQ;   (K, V) -> dV and dK
//
// so that the backward reads Q and dO once, K and V twice.
//
// Where a wave owns rows instead (cotten_wide32.hip), it reads all of the operand images of W, 98 KB, for every 16 rows:
// as many LDS cycles as the products take on the matrix cores, and the images leave LDS for one workgroup per compute
// unit; and its backward, in two roles, reads every tensor twice.  512 slices x 200 rows, fp32 d_h = 128, forward / backward:
// 60 / 155 -> 53 / 124 us (3.1 and 2.6 TB/s of what has to move).  What bounds these: the waves of a SIMD are two, and staging
// (vector units), LDS reads and products of a wave follow one another.  Cycles of a round of the backward, 32 rows: 4.1 k for
// S, 6.3 k for dS and dQ, of which the matrix cores need 1.5 k and 3.1 k; 1.5 k + 2.5 k from one walk to the next.  The forward has
// four waves per workgroup and two of these on a compute unit, which overlap (eight waves and one workgroup: 61 us); the
// backward's accumulators and operands take the registers of eight waves (four: 67 spilled, 155 us).  Staging cut into pieces
// among the products, without branches: 69 / 164 (registers, and all waves in the same phase).
#include "cotten_launch.h"
#include "cotten_mfma_core.h"

namespace cotten {
namespace {
namespace columns {

using namespace mfma;

extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

// How a format's tiles are read 32 columns at a time.
//   rows()   operand of a 32x32x16 product that contracts over the 16 rows of a tile
//   own()    the 16 rows as the operand of a 16x16x32 product that contracts over 32 columns: lane (i16, g16)
//            holds eight columns column(g16, 0 .. 7) of row i16
//   a product over a group of 32 output columns leaves the lane with the same eight columns: value
//            4 nt + v of the pair out[nt][v]; place(nt, i16) is the output column of row i16 of operand nt
template <class F>
struct Cols;

template <>
struct Cols<F32x32> {
  typedef F32x32 F;
  typedef Pieces Frag;
  static __device__ __forceinline__ Frag rows(const unsigned char* tiles, int group, const Lane& L) {
    return F::rows_operand(tiles + group * F::kTileBytes, L);
  }
  static __device__ __forceinline__ Frag own(const unsigned char* tiles, int group, const Lane& L) {
    F::TileRows t;
    t.load(tiles + group * F::kTileBytes, L);
    return t.a;
  }
  static __device__ __forceinline__ void values(const Frag& x, float (&f)[8]) {
    F::TileRows t;
    t.a = x;
    t.unpack(f);
  }
  template <bool INF>
  static __device__ __forceinline__ Frag cut(const float (&f)[8]) {
    F::TileRows t;
    t.set<INF>(f);
    return t.a;
  }
  static __device__ __forceinline__ int column(int g16, int e) { return 16 * (e >> 2) + 4 * g16 + (e & 3); }
  static __device__ __forceinline__ int place(int nt, int i16) { return 16 * nt + i16; }
  // two independent chains of products side by side
  static __device__ __forceinline__ void mfma16(const Frag (&w)[2], const Frag& x, f32x4_t (&out)[2]) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) out[nt] = Bf16Elem::mfma16(w[nt].l, x.h, out[nt]);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) out[nt] = Bf16Elem::mfma16(w[nt].h, x.l, out[nt]);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) out[nt] = Bf16Elem::mfma16(w[nt].m, x.m, out[nt]);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) out[nt] = Bf16Elem::mfma16(w[nt].m, x.h, out[nt]);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) out[nt] = Bf16Elem::mfma16(w[nt].h, x.m, out[nt]);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) out[nt] = Bf16Elem::mfma16(w[nt].h, x.h, out[nt]);
  }
  // a product of two operands in two steps (see F32x32): what the second needs of an operand is its largest piece
  static __device__ __forceinline__ f32x16_t mfma32_small(const Frag& a, const Frag& b, f32x16_t c) { return F::mfma32_small(a, b, c); }
  typedef bf16x8_t Large;
  static __device__ __forceinline__ Large large(const Frag& a) { return a.h; }
  static __device__ __forceinline__ f32x16_t mfma32_large(Large a, Large b, f32x16_t c) { return Bf16Elem::mfma32(a, b, c); }
  static __device__ __forceinline__ int run_row(int j, const Lane& L) { return F::run_row(j, L); }
  static __device__ __forceinline__ int run_col(const Lane& L) { return F::run_col(L); }
};
template <class E>
struct Cols<Half64<E>> {
  typedef Half64<E> F;
  typedef typename F::v8_t Frag;
  static __device__ __forceinline__ Frag rows(const unsigned char* tiles, int group, const Lane& L) {
    return F::rows_operand(tiles + (group >> 1) * F::kTileBytes, L, 32 * (group & 1));
  }
  static __device__ __forceinline__ Frag own(const unsigned char* tiles, int group, const Lane& L) {
    return *reinterpret_cast<const Frag*>(tiles + (group >> 1) * F::kTileBytes + L.i16 * F::kTileStride + 64 * (group & 1) + 16 * L.g16);
  }
  static __device__ __forceinline__ void values(const Frag& x, float (&f)[8]) { F::unpack(__builtin_bit_cast(u32x4_t, x), f); }
  template <bool>
  static __device__ __forceinline__ Frag cut(const float (&f)[8]) { return __builtin_bit_cast(Frag, F::pack(f)); }
  static __device__ __forceinline__ int column(int g16, int e) { return 8 * g16 + e; }
  static __device__ __forceinline__ int place(int nt, int i16) { return 8 * (i16 >> 2) + 4 * nt + (i16 & 3); }
  static __device__ __forceinline__ void mfma16(const Frag (&w)[2], const Frag& x, f32x4_t (&out)[2]) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) out[nt] = E::mfma16(w[nt], x, out[nt]);
  }
  static __device__ __forceinline__ f32x16_t mfma32(const Frag& a, const Frag& b, f32x16_t c) { return E::mfma32(a, b, c); }
  static __device__ __forceinline__ int run_row(int j, const Lane& L) { return F::BlockAcc::run_row(j, L); }
  static __device__ __forceinline__ int run_col(const Lane& L) { return F::BlockAcc::run_col(L); }
};
template <class Base>
struct Cols<WithElu1<Base>> : Cols<Base> {};

// A workgroup has one, two or four waves per group of 32 columns: a round has as many tiles of x and of y, and the
// waves of a group share its work (`part`).
template <class F, int P, int WAVES>
struct Lds {
  static constexpr int D = P * F::D, kGroups = D / 32, kParts = WAVES / kGroups;
  static constexpr int kRound = TR * kParts;                           // rows of x and of y in a round
  static constexpr int kY = P * F::kTileBytes, kPair = 2 * kY;         // [x pieces | y pieces] of 16 rows
  static constexpr int kBuffer = kParts * kPair;
  static constexpr int kLd = D + 4, kMatrix = D * kLd * 4;             // a state, between two walks
  static constexpr int kTiles = 2 * kBuffer > kMatrix ? 2 * kBuffer : kMatrix;
  static constexpr int kFactors = kTiles;                              // [buffer][row of a round, of one without y]
  static constexpr int kDots = kFactors + 2 * 2 * kRound * 4;          // [buffer][group][row of a round]
  static constexpr int kLive = kDots + 2 * kGroups * kRound * 4;       // [buffer][wave]
  static constexpr int kBytes = kLive + 2 * WAVES * 4;
  static_assert(kGroups == 4 && (kParts == 1 || kParts == 2 || kParts == 4), "shape");
};

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
  float scale, eps;
  const float* slice_scale;
  float* kept;  // forward: S of every slice, or nullptr
  float* dlog;  // backward: d loss / d log(scale) of every slice, or nullptr
  Strides st;
};

// What becomes of the rows of a round on their way to LDS, and who brings them there (eight rows of a tensor at a time).
enum Stage {
  kMapped,  // x: xhat or phi(x), the first half of the waves;  y as it is, the second half
  kRaw,     // x as it is (phi(x) under ELU + 1) and y as it is, both the first half of the waves
  kRawX,    // x alone, all waves: twice as many rows
};

// A walk over the rows of a tensor pair: the wave's share of the round after the staged one is on its way in
// registers.  Rows that do not take part are never fetched.
template <class F, int P, int WAVES, int STAGE>
struct Walk {
  typedef Lds<F, P, WAVES> Map;
  static constexpr bool kBoth = STAGE == kRaw;  // a wave brings x and y, or nothing
  static constexpr int kRows = STAGE == kRawX ? 2 * Map::kRound : Map::kRound, kUnits = kBoth ? 2 : 1;
  __amdgpu_buffer_rsrc_t src[kUnits];
  const uint8_t* mask;
  int stride, end, slot;  // `slot`: the wave's first row of a round
  bool is_x, idle;
  u32x4_t raw[kUnits][P];
  bool live, next_live;  // the row takes part: that of `raw`, that of the round behind it
  int next_row;          // of the workgroup, of the round behind `raw`

  __device__ __forceinline__ Walk(const unsigned char* X, const unsigned char* Y, int N, RowAddr addr,
                                  const uint8_t* m, const Lane& L)
      : mask(m), stride(addr.stride), end(N) {
    const bool first_half = L.wave < WAVES / 2;
    is_x = STAGE == kRawX || first_half;
    idle = kBoth && !first_half;
    slot = 8 * (STAGE == kRawX ? L.wave : L.wave & (WAVES / 2 - 1));
    if constexpr (kBoth) {
      src[0] = Buffers(X, N, addr).r;
      src[1] = Buffers(Y, N, addr).r;
    } else {
      src[0] = Buffers(is_x ? X : Y, N, addr).r;
    }
  }
  __device__ __forceinline__ bool row_live(int row0, const Lane& L) const {
    const int row = row0 + slot + L.r8;
    return row < end && (mask == nullptr || mask[row] != 0);
  }
  __device__ __forceinline__ void load(int row0, const Lane& L) {
    const uint32_t off = live ? static_cast<uint32_t>(row0 + slot + L.r8) * stride + L.ch * 16 : kOutOfBuffer;
#pragma unroll
    for (int u = 0; u < kUnits; ++u)
#pragma unroll
      for (int c = 0; c < P; ++c) raw[u][c] = __builtin_amdgcn_raw_buffer_load_b128(src[u], off + c * kRowBytes, 0, 0);
  }
  // asks for the round at `begin`
  __device__ __forceinline__ void start(int begin, const Lane& L) {
    if (idle) return;
    live = row_live(begin, L);
    load(begin, L);
    next_row = begin + kRows;
    next_live = row_live(next_row, L);
  }
  // the round on its way into LDS buffer `buffer`, and asks for the next one
  __device__ __forceinline__ void advance(int buffer, float eps, const Lane& L) {
    if (idle) return;
    unsigned char* tiles = smem + buffer * Map::kBuffer;
    if (kBoth) {
      tiles += slot / TR * Map::kPair;
      stage_x(tiles, buffer, eps, L);
      stage_y(raw[kUnits - 1], tiles + Map::kY, L);
    } else if (STAGE == kRawX) {  // (tile by tile, where x and y lie otherwise)
      stage_x(tiles + slot / TR * Map::kY, buffer, eps, L);
    } else {
      tiles += slot / TR * Map::kPair;
      if (is_x) stage_x(tiles, buffer, eps, L);
      else stage_y(raw[0], tiles + Map::kY, L);
    }
    live = next_live;
    load(next_row, L);
    next_row += kRows;
    next_live = row_live(next_row, L);
  }

  __device__ __forceinline__ void stage_x(unsigned char* tiles, int buffer, float eps, const Lane& L) {
    const bool any = __builtin_amdgcn_ballot_w64(live) != 0;
    if (L.lane == 0) reinterpret_cast<int*>(smem + Map::kLive)[WAVES * buffer + L.wave] = any;
    float top = 0.0f;  // (phi(x) is infinite where x is)
    if (F::kMap == kMapElu1) {
#pragma unroll
      for (int c = 0; c < P; ++c) top = F::largest_raw(raw[0][c], top);
    }
    write_pieces<F>(top, [&](auto inf) {
      float f[P][F::EPL];
      float ss = 0.0f;
#pragma unroll
      for (int c = 0; c < P; ++c) {
        F::unpack(raw[0][c], f[c]);
#pragma unroll
        for (int i = 0; i < F::EPL; ++i) ss += f[c][i] * f[c][i];
      }
      const float inv = F::kMap == kMapElu1 ? 1.0f : inv_norm_or_zero(row_sum8(ss), eps, live);
      if (L.ch == 0)
        reinterpret_cast<float*>(smem + Map::kFactors)[2 * Map::kRound * buffer + slot + L.r8] = live ? inv : -1.0f;
#pragma unroll
      for (int c = 0; c < P; ++c) {
        if (F::kMap == kMapElu1) {
#pragma unroll
          for (int i = 0; i < F::EPL; ++i) f[c][i] = elu1_or_zero(f[c][i], live);
        } else if (STAGE == kMapped) {
#pragma unroll
          for (int i = 0; i < F::EPL; ++i) f[c][i] *= inv;
        }
        F::template put<decltype(inf)::value>(tiles + c * F::kTileBytes, (slot & (TR - 1)) + L.r8, L.ch, f[c]);
      }
    });
  }
  __device__ __forceinline__ void stage_y(const u32x4_t (&y)[P], unsigned char* tiles, const Lane& L) {
    float top = 0.0f;
#pragma unroll
    for (int c = 0; c < P; ++c) top = F::largest_raw(y[c], top);
    write_pieces<F>(top, [&](auto inf) {
#pragma unroll
      for (int c = 0; c < P; ++c)
        F::template put_raw<decltype(inf)::value>(tiles + c * F::kTileBytes, (slot & (TR - 1)) + L.r8, L.ch, y[c]);
    });
  }
};

// The rounds begin .. end-1 of a walk that has been started: round(buffer, row0) is called with the round in LDS
// buffer `buffer`, after(buffer, row0) one barrier behind it.  Half of the waves stage the next round (vector units) ahead
// of their products (matrix cores), the others behind them.
template <int WAVES, class W, class Round, class After>
__device__ __forceinline__ void rounds(W& walk, int begin, int end, float eps, const Lane& L, Round&& round,
                                       After&& after) {
  if (begin >= end) return;
  walk.advance(0, eps, L);
  int buffer = 0;
#pragma unroll 1
  for (int r0 = begin; r0 < end; r0 += W::kRows) {
    __syncthreads();  // the round is staged; nobody reads the other buffer any more
    if (r0 > begin) after(buffer ^ 1, r0 - W::kRows);
    const bool more = r0 + W::kRows < end;
    if (more && L.wave < WAVES / 2) walk.advance(buffer ^ 1, eps, L);
    round(buffer, r0);
    if (more && L.wave >= WAVES / 2) walk.advance(buffer ^ 1, eps, L);
    buffer ^= 1;
  }
  __syncthreads();
  after(buffer ^ 1, begin + (end - begin - 1) / W::kRows * W::kRows);
}

// ---- states -----------------------------------------------------------------------------------------

// The wave's blocks of a state: columns 32 p .. of x against 32 (q0 + j) .. of y.  fp32: the products of
// a round are summed up on their own, small ones first, and then added to what there is: few roundings at its size.
template <class F, int P, int WAVES>
struct State {
  typedef Lds<F, P, WAVES> Map;
  typedef Cols<F> C;
  static constexpr int kBlocks = Map::kGroups / Map::kParts;
  f32x16_t v[kBlocks];
  int p, q0;
  __device__ __forceinline__ explicit State(const Lane& L) : p(L.wave / Map::kParts), q0(L.wave % Map::kParts * kBlocks) {
#pragma unroll
    for (int j = 0; j < kBlocks; ++j)
#pragma unroll
      for (int i = 0; i < 16; ++i) v[j][i] = 0.0f;
  }
  __device__ __forceinline__ void add(int buffer, const Lane& L) {
    constexpr int T = Map::kParts;
    const unsigned char* tiles = smem + buffer * Map::kBuffer;
    if constexpr (!F::kPieces) {
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const typename C::Frag x = C::rows(tiles + t * Map::kPair, p, L);
#pragma unroll
        for (int j = 0; j < kBlocks; ++j) v[j] = C::mfma32(x, C::rows(tiles + t * Map::kPair + Map::kY, q0 + j, L), v[j]);
      }
    } else {
      add_pieces(tiles, L);
    }
  }
  __device__ __forceinline__ void add_pieces(const unsigned char* tiles, const Lane& L) {
    constexpr int T = Map::kParts;
    f32x16_t sum[kBlocks];
    typename C::Large x_large[T], y_large[T][kBlocks];
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const typename C::Frag x = C::rows(tiles + t * Map::kPair, p, L);
      x_large[t] = C::large(x);
#pragma unroll
      for (int j = 0; j < kBlocks; ++j) {
        if (t == 0) {
#pragma unroll
          for (int i = 0; i < 16; ++i) sum[j][i] = 0.0f;
        }
        const typename C::Frag y = C::rows(tiles + t * Map::kPair + Map::kY, q0 + j, L);
        y_large[t][j] = C::large(y);
        sum[j] = C::mfma32_small(x, y, sum[j]);
        if (t < T - 1) continue;
#pragma unroll
        for (int u = 0; u < T; ++u) sum[j] = C::mfma32_large(x_large[u], y_large[u][j], sum[j]);
#pragma unroll
        for (int i = 0; i < 16; ++i) v[j][i] += sum[j][i];
      }
    }
  }
  // into the matrix in LDS, row-major
  __device__ __forceinline__ void write(const Lane& L) const {
    float* M = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int j = 0; j < kBlocks; ++j)
#pragma unroll
      for (int run = 0; run < 4; ++run) {
        float* at = M + (32 * p + C::run_row(run, L)) * Map::kLd + 32 * (q0 + j) + C::run_col(L);
#pragma unroll
        for (int i = 0; i < 4; ++i) at[i * Map::kLd] = v[j][4 * run + i];
      }
  }
};

// The wave's 32 columns of products with scale * M, as operands.
template <class F, int P, int WAVES>
struct Weights {
  typedef Lds<F, P, WAVES> Map;
  typedef Cols<F> C;
  typename C::Frag w[Map::kGroups][2];
  // natural: T = Y M^T, output column n is row n of M.  Otherwise T = X M, output column n is column n.
  __device__ __forceinline__ void load(int group, float scale, bool natural, const Lane& L) {
    const float* M = reinterpret_cast<const float*>(smem);
    float f[Map::kGroups][2][8], top = 0.0f;
    if (natural) {
#pragma unroll
      for (int ks = 0; ks < Map::kGroups; ++ks)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
          for (int e = 0; e < 8; ++e)
            f[ks][nt][e] = M[(32 * group + C::place(nt, L.i16)) * Map::kLd + 32 * ks + C::column(L.g16, e)];
    } else {
#pragma unroll
      for (int ks = 0; ks < Map::kGroups; ++ks)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
          for (int e = 0; e < 8; ++e)
            f[ks][nt][e] = M[(32 * ks + C::column(L.g16, e)) * Map::kLd + 32 * group + C::place(nt, L.i16)];
    }
#pragma unroll
    for (int ks = 0; ks < Map::kGroups; ++ks)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
#pragma unroll
        for (int e = 0; e < 8; ++e) f[ks][nt][e] *= scale;
        if (F::kPieces) top = largest(f[ks][nt], top);
      }
    write_pieces<F>(top, [&](auto inf) {
#pragma unroll
      for (int ks = 0; ks < Map::kGroups; ++ks)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) w[ks][nt] = C::template cut<decltype(inf)::value>(f[ks][nt]);
    });
  }
  // the wave's columns of (rows of the tile) x W
  __device__ __forceinline__ void apply(const unsigned char* tiles, const Lane& L, float (&o)[8]) const {
    f32x4_t out[2];
    out[0] = out[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < Map::kGroups; ++ks) C::mfma16(w[ks], C::own(tiles, ks, L), out);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int v = 0; v < 4; ++v) o[4 * nt + v] = out[nt][v];
  }
};

// The state of all waves into the matrix in LDS.  Begins and ends with a barrier; the tiles are overwritten.
template <class S>
__device__ __forceinline__ void publish(const S& state, const Lane& L) {
  __syncthreads();
  state.write(L);
  __syncthreads();
}

// ---- rows of results ----------------------------------------------------------------------------------

// The lane's eight columns of a row of the wave's 32.
template <class F>
__device__ __forceinline__ void store_columns(unsigned char* out, int group, int row, int end, int stride, const Lane& L,
                                              const float (&o)[8]) {
  if (row >= end) return;
  if constexpr (F::kPieces) {
    store_product_row<F, kStoreStreamed>(out + group * kRowBytes, row, RowAddr{stride, kRowBytes}, L, o);
  } else {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(out, 0, 0x7fffffff, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b128(F::pack(o), r, static_cast<uint32_t>(row) * stride + 64 * group + 16 * L.g16, 0,
                                           kStoreStreamed);
  }
}

// Rows first .. last-1 of a result that are zeros.
template <class F, int P, int THREADS>
__device__ __forceinline__ void store_zero_rows(unsigned char* out, int last, int stride) {
  constexpr int kChunks = P * kRowBytes / 16;
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(out, 0, 0x7fffffff, 0x00020000);
#pragma unroll 1
  for (int e = threadIdx.x; e < last * kChunks; e += THREADS)
    __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{0, 0, 0, 0}, r,
                                           static_cast<uint32_t>(e / kChunks) * stride + e % kChunks * 16, 0,
                                           kStoreStreamed);
}

// A tile of dQ or dK between its product and its rows' dot products: the lane's columns of g and of the x rows.
struct Projected {
  float g[8], x[8];
  float inv;  // 1/r (1 under ELU + 1); below zero: the row does not take part
};

// sum over the lane's columns of (mapped x) . g, to the row's place in LDS
__device__ __forceinline__ void publish_dot(const Projected& t, float* place, const Lane& L) {
  float dot = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) dot += t.x[i] * t.g[i];
  dot = row_sum_groups(dot, L);
  if (L.g16 == 0) place[L.i16] = dot;
}

// g <- J g, J the derivative of the map
template <class F>
__device__ __forceinline__ void finish(Projected& t, float dot) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if (F::kMap == kMapElu1) t.g[i] *= fminf(t.x[i], 1.0f);
    else t.g[i] = (t.g[i] - t.x[i] * dot) * t.inv;
    t.g[i] = t.inv < 0.0f ? 0.0f : t.g[i];
  }
}

// First row at which a key is valid, down to a multiple of 16 (N if there is none): a left-padded history is walked
// from there.  Every wave looks for itself, 512 rows at a time.
__device__ __forceinline__ int first_live_tile(const uint8_t* __restrict__ m, int N, const Lane& L) {
  if (m == nullptr) return 0;
#pragma unroll 1
  for (int row0 = 0; row0 < N; row0 += 512) {
    uint64_t set[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = row0 + 64 * i + L.lane;
      set[i] = __builtin_amdgcn_ballot_w64(row < N && m[row < N ? row : 0] != 0);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (set[i] != 0) return (row0 + 64 * i + __builtin_ctzll(set[i])) & ~(TR - 1);
  }
  return N;
}

// The round in `buffer` has rows that take part.
template <class Map, int WAVES>
__device__ __forceinline__ bool round_live(int buffer) {
  const int* live = reinterpret_cast<const int*>(smem + Map::kLive) + WAVES * buffer;
  int any = 0;
#pragma unroll
  for (int w = 0; w < WAVES / 2; ++w) any |= live[w];
  return __builtin_amdgcn_readfirstlane(any) != 0;
}

// ---- kernels -------------------------------------------------------------------------------------------

// S of the slice over its keys.
template <class F, int P, int WAVES>
__device__ __forceinline__ void key_state(State<F, P, WAVES>& s, const Args& a, size_t base, const uint8_t* keys, int begin,
                                          const Lane& L) {
  Walk<F, P, WAVES, kMapped> kv(a.K + base, a.V + base, a.N, a.st.row, keys, L);
  kv.start(begin, L);
  rounds<WAVES>(kv, begin, a.N, a.eps, L, [&](int buffer, int) {
    if (round_live<Lds<F, P, WAVES>, WAVES>(buffer)) s.add(buffer, L);
  }, [](int, int) {});
}

template <class F, int P, int WAVES, int PER_SIMD>
__global__ __launch_bounds__(64 * WAVES, PER_SIMD) void columns_fwd_kernel(const Args a) {
  typedef Lds<F, P, WAVES> Map;
  const Lane L;
  const int group = L.wave % Map::kGroups, part = L.wave / Map::kGroups;
  const int bh = blockIdx.x, N = a.N;
  const size_t base = a.st.slice_base(bh, a.H);
  const uint8_t* keys = a.mask == nullptr ? nullptr : a.mask + static_cast<size_t>(bh / a.H) * N;
  const float scale = a.slice_scale != nullptr ? a.slice_scale[bh] : a.scale;
  State<F, P, WAVES> s(L);
  key_state<F, P, WAVES>(s, a, base, keys, first_live_tile(keys, N, L), L);
  Walk<F, P, WAVES, kRawX> q(a.Q + base, nullptr, N, a.st.row, nullptr, L);
  q.start(0, L);
  publish(s, L);
  if (a.kept != nullptr) {
    constexpr int D = Map::D;
    float* out = a.kept + static_cast<size_t>(bh) * D * D;
    for (int e = threadIdx.x; e < D * D / 4; e += 64 * WAVES)
      *reinterpret_cast<f32x4_t*>(out + 4 * e) =
          *reinterpret_cast<const f32x4_t*>(reinterpret_cast<const float*>(smem) + 4 * e / D * Map::kLd + 4 * e % D);
  }
  Weights<F, P, WAVES> W;
  W.load(group, scale, false, L);
  __syncthreads();
  rounds<WAVES>(q, 0, N, a.eps, L, [&](int buffer, int row0) {
    const float* factors = reinterpret_cast<const float*>(smem + Map::kFactors) + 2 * Map::kRound * buffer;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int t = part + i * Map::kParts;
      if (row0 + t * TR >= N) continue;
      float o[8];
      W.apply(smem + buffer * Map::kBuffer + t * Map::kY, L, o);
      const float inv = factors[t * TR + L.i16];
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] *= inv;
      store_columns<F>(a.O + base, group, row0 + t * TR + L.i16, N, a.st.row.stride, L, o);
    }
  }, [](int, int) {});
}

// DLOG: <S, dS> from the accumulators of both, which 16-bit rows take for the gradient of the scale; fp32 rows sum up the
// dot products of the rows.
template <class F, int P, int WAVES, int PER_SIMD, bool DLOG>
__global__ __launch_bounds__(64 * WAVES, PER_SIMD) void columns_bwd_kernel(const Args a) {
  constexpr int kShare = Lds<F, P, WAVES>::kParts / 2;  // waves of a group that share dV (dK)
  typedef Lds<F, P, WAVES> Map;
  typedef Cols<F> C;
  const Lane L;
  const int bh = blockIdx.x, N = a.N, stride = a.st.row.stride;
  const size_t base = a.st.slice_base(bh, a.H);
  const uint8_t* keys = a.mask == nullptr ? nullptr : a.mask + static_cast<size_t>(bh / a.H) * N;
  const float scale = a.slice_scale != nullptr ? a.slice_scale[bh] : a.scale;
  const int group = L.wave % Map::kGroups, part = L.wave / Map::kGroups;
  const int begin = first_live_tile(keys, N, L);
  const bool want_dots = F::kMap != kMapElu1 || (F::kPieces && a.dlog != nullptr);
  float* all_dots = reinterpret_cast<float*>(smem + Map::kDots);
  const auto dots_of = [&](int buffer, int g) { return all_dots + (buffer * Map::kGroups + g) * Map::kRound; };
  const auto row_dot = [&](int buffer, int row) {
    float d = dots_of(buffer, 0)[row];
#pragma unroll
    for (int g = 1; g < Map::kGroups; ++g) d += dots_of(buffer, g)[row];
    return d;
  };
  const auto factor_of = [&](int buffer, int row) {
    return reinterpret_cast<const float*>(smem + Map::kFactors)[2 * Map::kRound * buffer + row];
  };
  State<F, P, WAVES> s(L);
  key_state<F, P, WAVES>(s, a, base, keys, begin, L);
  State<F, P, WAVES> ds(L);
  Weights<F, P, WAVES> W;
  {  // dS and dQ: a wave has one of the two tiles of a round
    Walk<F, P, WAVES, kMapped> qg(a.Q + base, a.dO + base, N, a.st.row, nullptr, L);
    qg.start(0, L);
    publish(s, L);
    W.load(group, scale, true, L);
    __syncthreads();
    Projected t;
    float dlog = 0.0f;
    rounds<WAVES>(qg, 0, N, a.eps, L, [&](int buffer, int) {
      const unsigned char* tiles = smem + buffer * Map::kBuffer + part * Map::kPair;
      ds.add(buffer, L);
      W.apply(tiles + Map::kY, L, t.g);
      C::values(C::own(tiles, group, L), t.x);
      t.inv = factor_of(buffer, part * TR + L.i16);
      if (want_dots) publish_dot(t, dots_of(buffer, group) + part * TR, L);
    }, [&](int buffer, int row0) {
      const int row = row0 + part * TR + L.i16;
      const float dot = want_dots ? row_dot(buffer, part * TR + L.i16) : 0.0f;
      if (row < N) dlog += dot;
      finish<F>(t, dot);
      store_columns<F>(a.dQ + base, group, row, N, stride, L, t.g);
    });
    if (F::kPieces ? a.dlog != nullptr : DLOG) {  // in a fixed order
      float sum = 0.0f;
      if constexpr (F::kPieces) {  // sum_i dO_i . O_i = sum_i qhat_i . (scale dO_i S^T)
        sum = group == 0 && L.g16 == 0 ? dlog : 0.0f;
      } else {
#pragma unroll
        for (int j = 0; j < State<F, P, WAVES>::kBlocks; ++j)
#pragma unroll
          for (int i = 0; i < 16; ++i) sum += s.v[j][i] * ds.v[j][i];
      }
      sum = wave_sum(sum);
      __syncthreads();
      if (L.lane == 0) all_dots[L.wave] = sum;
      __syncthreads();
      if (threadIdx.x == 0) {
        float total = 0.0f;
        for (int w = 0; w < WAVES; ++w) total += all_dots[w];
        a.dlog[bh] = F::kPieces ? total : total * scale;
      }
    }
  }
  {  // dV = scale khat dS (the first half of the waves, which also stage the rows) and dK from scale v dS^T (the others)
    const bool plain = part < kShare;
    const int first = plain ? part : part - kShare;
    Walk<F, P, WAVES, kRaw> kv(a.K + base, a.V + base, N, a.st.row, keys, L);
    kv.start(begin, L);
    publish(ds, L);
    W.load(group, scale, !plain, L);
    __syncthreads();
    Projected t[2];
    rounds<WAVES>(kv, begin, N, a.eps, L, [&](int buffer, int row0) {
      const unsigned char* tiles = smem + buffer * Map::kBuffer;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int at = (first + i * kShare) * TR;  // row of the round
        const unsigned char* pair = tiles + at / TR * Map::kPair;
        const float inv = factor_of(buffer, at + L.i16);
        if (plain) {
          float o[8];
          W.apply(pair, L, o);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = inv < 0.0f ? 0.0f : o[e] * inv;
          store_columns<F>(a.dV + base, group, row0 + at + L.i16, N, stride, L, o);
          continue;
        }
        W.apply(pair + Map::kY, L, t[i].g);
        C::values(C::own(pair, group, L), t[i].x);
        t[i].inv = inv;
        if (F::kMap == kMapElu1) continue;
#pragma unroll
        for (int e = 0; e < 8; ++e) t[i].x[e] *= t[i].inv;  // (below zero: the row's results are dropped)
        publish_dot(t[i], dots_of(buffer, group) + at, L);
      }
    }, [&](int buffer, int row0) {
      if (plain) return;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int at = (first + i * kShare) * TR;
        finish<F>(t[i], F::kMap != kMapElu1 ? row_dot(buffer, at + L.i16) : 0.0f);
        store_columns<F>(a.dK + base, group, row0 + at + L.i16, N, stride, L, t[i].g);
      }
    });
  }
  store_zero_rows<F, P, 64 * WAVES>(a.dV + base, begin, stride);
  store_zero_rows<F, P, 64 * WAVES>(a.dK + base, begin, stride);
}

// ---- host side -------------------------------------------------------------------------------------------

constexpr long kUnits = 256;

template <class Kernel>
hipError_t launch(Kernel kernel, int waves, int lds, const Problem& p, const Args& a) {
  const hipError_t err = grant_dynamic_lds(reinterpret_cast<const void*>(kernel), lds);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(p.B) * p.H), dim3(64 * waves), lds, p.stream, a);
  return hipGetLastError();
}

hipError_t run32(const Problem& p, const Args& a, bool bwd) {
  const auto go = [&](auto f) {
    typedef decltype(f) F;
    constexpr int lds_fwd = Lds<F, 4, 4>::kBytes, lds_bwd = Lds<F, 4, 8>::kBytes;
    static_assert(lds_fwd <= 80 * 1024 && lds_bwd <= 160 * 1024, "two workgroups per compute unit, and one");
    return bwd ? launch(columns_bwd_kernel<F, 4, 8, 2, false>, 8, lds_bwd, p, a)
               : launch(columns_fwd_kernel<F, 4, 4, 2>, 4, lds_fwd, p, a);
  };
  return p.feature_map == kMapElu1 ? go(WithElu1<F32x32>{}) : go(F32x32{});
}

// 16-bit rows, backward: eight waves, two workgroups per compute unit, where there are more slices than units, sixteen
// otherwise and where the accumulators of S are kept for <S, dS> (registers).  bf16 d_h = 128, sixteen and eight, us:
// 256 x 400 47.7, 58.2;  300 x 300 61.8, 51.4;  512 x 300 77.9, 65.6;  512 x 500 120, 115;  700 x 500 162, 165.
template <class F>
hipError_t run16(const Problem& p, const Args& a) {
  constexpr int lds8 = Lds<F, 2, 8>::kBytes, lds16 = Lds<F, 2, 16>::kBytes;
  static_assert(lds8 <= 80 * 1024 && lds16 <= 160 * 1024, "two workgroups per compute unit, and one");
  if (a.dlog != nullptr) return launch(columns_bwd_kernel<F, 2, 16, 4, true>, 16, lds16, p, a);
  if (static_cast<long>(p.B) * p.H > kUnits) return launch(columns_bwd_kernel<F, 2, 8, 4, false>, 8, lds8, p, a);
  return launch(columns_bwd_kernel<F, 2, 16, 4, false>, 16, lds16, p, a);
}

}  // namespace columns
}  // namespace

// fp32 rows of 512 bytes.  The kernels of cotten_wide32.hip have one workgroup (backward: two) of eight waves per slice
// and compute unit; they stay where these fit the chip at once, and these kernels take over from there (forward / backward, us,
// those and these):  128 slices x 200 rows 26.6 / 39.7, 36.5 / 58.8;  192: 30.2 / 73.4, 40.2 / 60.6;  256: 33.4 / 76.8, 41.5 /
// 62.3;  300: 50.0 / 104, 48.0 / 104;  512: 60.4 / 155, 53.0 / 123;  512 x 100 36.5 / 95.9, 31.6 / 77.3;  512 x 20 19.9 / 61.6, 11.6 /
// 32.8;  512 x 700 163 / 415, 164 / 368;  256 x 1000 118 / 283, 181 / 277.  Forwards of longer sequences stay there, one
// workgroup per compute unit in rounds of 256:  280 x 300 57.5, 61.7;  280 x 700 121, 136;  512 x 300 65.1, 65.5;  519 x 700 193, 218;  640 x 500
// 158, 173 - but 900 x 300 132, 127, and 900 x 400 171, 164.  (Errors against float64 1.9e-7, here 2.1e-7.)  Backwards of 258 ... 384 slices and more
// than 256 rows are faster there too, 280 x 400 159, 170, 280 x 1000 390, 416, but less exact, dK of 300 x 1000 2.2e-7, 2.1e-7: not them.
// 16-bit rows of 256 bytes, backward: against the kernels of cotten_wide.hip, which keep the tiles of up to 256 rows in
// registers and walk longer sequences three times (us, those and these):  1024 slices x 200 rows 94.6, 99.6;  100 x 300 31.5,
// 34.2;  180 x 300 34.8, 36.2;  180 x 400 45.3, 43.8;  256 x 300 38.2, 37.2;  512 x 300 85.0, 65.6;  512 x 400 117, 87;  256 x 800 130, 96;
// 200 x 1800 255, 192.  (Their forward stays: 512 x 400 37, 39.)
bool columns_apply(const Problem& p, bool bwd) {
  const long slices = static_cast<long>(p.B) * p.H;
  if (p.D != 128) return false;
  if (p.dtype != 0) return bwd && (p.N > 384 || (p.N > 256 && slices >= columns::kUnits));
  if (bwd) return 2 * slices > columns::kUnits;
  return slices > columns::kUnits && (p.N <= 256 || (slices - 1) / columns::kUnits == 3);
}

hipError_t launch_columns(const Problem& p, bool bwd) {
  using namespace columns;
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
  a.scale = p.scale;
  a.eps = p.eps;
  a.slice_scale = p.slice_scale;
  a.kept = p.saved_state;
  a.dlog = p.dlog_scale;
  const long long e = p.elem_bytes();
  a.st = Strides{p.stride_batch * e, p.stride_head * e,
                 RowAddr{static_cast<int>(p.stride_row * e), static_cast<int>(p.D * e)}};
  if (p.dtype == 0) return run32(p, a, bwd);
  if (!bwd) return hipErrorInvalidValue;
  if (p.feature_map == kMapElu1) return p.dtype == 1 ? run16<WithElu1<Bf16x64>>(p, a) : run16<WithElu1<F16x64>>(p, a);
  return p.dtype == 1 ? run16<Bf16x64>(p, a) : run16<F16x64>(p, a);
}

}  // namespace cotten
