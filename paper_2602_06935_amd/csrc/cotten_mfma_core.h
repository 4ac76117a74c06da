// Device code shared by the MFMA kernels: rows in pieces of 128 bytes (16-bit d_h = 64, fp32 d_h = 32):
// lane geometry, the two element formats with their MFMA products, tile loads through
// buffer resources, staging into LDS tiles, and the epilogue helpers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace cotten {
namespace mfma {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

constexpr int TR = 16;               // rows per wave tile
constexpr int kRowBytes = 128;       // bytes of one tile row: d_h elements, or d_h/2 elements
                                     // followed by zeros (half-width rows)
constexpr int kTileStride = 144;     // bytes per row of an LDS tile (128 + 16 of padding)
constexpr int kTileBytes = TR * kTileStride;

// Sum over the 8 consecutive lanes that share one row, by lane-permuting adds (no LDS).
__device__ __forceinline__ float row_sum8(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));   // lane ^ 1
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true));   // lane ^ 2
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xF, 0xF, true));  // other quad of the 8
  return x;
}

// 1/sqrt(ss + eps) for a live row (hardware reciprocal square root, about 1 ulp), 0 otherwise.
// (MARK: -0 instead, see zero_masked.)
template <bool MARK = false>
__device__ __forceinline__ float inv_norm_or_zero(float ss, float eps, bool live) {
  return live ? __builtin_amdgcn_rsqf(ss + eps) : MARK ? -0.0f : 0.0f;
}

// dK and dV rows of masked keys are zeros by selection: as products of zero rows they would be NaN where the state or a
// later row is not finite.  The rows are told by their 1/r, -0, which reaches the layout of the products anyway (+0: a
// row that takes part and whose square sum overflows).
__device__ __forceinline__ bool is_masked(float inv_r) { return __builtin_bit_cast(uint32_t, inv_r) == 0x80000000u; }
template <int N>
__device__ __forceinline__ void zero_masked(float inv_r, float (&dk)[N], float (&dv)[N]) {
  if (is_masked(inv_r)) {  // (one branch over both: selects took 1 % of a causal backward)
#pragma unroll
    for (int i = 0; i < N; ++i) dk[i] = dv[i] = 0.0f;
  }
}

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  bf16x2_t v;
  v[0] = static_cast<__bf16>(lo);
  v[1] = static_cast<__bf16>(hi);
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ f32x4_t quad(const f32x16_t& a, int j) {
  return f32x4_t{a[4 * j], a[4 * j + 1], a[4 * j + 2], a[4 * j + 3]};
}

// Lane geometry shared by every pass.
struct Lane {
  int lane, wave;
  int r8, ch;    // load layout: tile rows r8 and r8+8, bytes 16*ch .. 16*ch+15 of the row
  int i16, g16;  // MFMA 16-lane groups: lane%16, lane/16
  __device__ __forceinline__ Lane() {
    set(threadIdx.x & 63);
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: lives in a scalar register
  }
  // The same geometry, recomputed from scratch where it is used: in a long kernel this keeps
  // the per-lane offsets derived from it from being carried (and spilled) across phases.
  __device__ __forceinline__ Lane again() const {
    Lane l = *this;
    int id = lane;
    asm volatile("" : "+v"(id));
    l.set(id);
    return l;
  }
  __device__ __forceinline__ void set(int id) {
    lane = id;
    r8 = lane >> 3;
    ch = lane & 7;
    i16 = lane & 15;
    g16 = lane >> 4;
  }
};

// ---- the two element formats ----------------------------------------------------------
//
// Common vocabulary of a format F:
//   F::D                  head dimension;  F::EPL = D/8 elements per lane in the load layout
//   F::unpack / F::pack   128-bit register group <-> EPL floats
//   F::Acc                accumulators of one D x D state per wave, with mfma() and the
//                         column-major image R[n*(D+4)+m] used for the cross-wave sum
//   F::Operand            a D x D matrix W held in registers for apply products, loaded from
//                         an LDS image op[n][k] (k contiguous); F::apply(tile, W, out)
//   F::write_image        builds such images from a reduced state

// The two 16-bit element types of the d_h = 64 format: how a pair sits in a 32-bit word, and
// the matrix-core and transposing-read instructions of the type.
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));

struct Bf16Elem {
  static constexpr bool kFloatRange = true;  // (nearly) the exponents of a float
  typedef bf16x8_t v8;
  typedef bf16x4_t v4;
  static __device__ __forceinline__ float lo(uint32_t w) { return __uint_as_float(w << 16); }
  static __device__ __forceinline__ float hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
  static __device__ __forceinline__ uint32_t pack2(float a, float b) { return pack_bf16(a, b); }
  static __device__ __forceinline__ f32x16_t mfma32(v8 a, v8 b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ f32x4_t mfma16(v8 a, v8 b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ v4 read_tr(const unsigned char* p) {
    typedef v4 __attribute__((address_space(3))) * lds_v4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_v4)(p));
  }
  // 16x16x16: A lane (i = lane%16, k = 4*(lane/16) + e), B lane (j = lane%16, same k): the k
  // a lane holds is the row group it holds of a 16x16 result, so a result (rounded) can be fed
  // back as the B operand without moving between lanes
  static __device__ __forceinline__ f32x4_t mfma_k16(v4 a, v4 b, f32x4_t c) {
    typedef short s16x4_t __attribute__((ext_vector_type(4)));
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, a),
                                                     __builtin_bit_cast(s16x4_t, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ v4 pack4(f32x4_t x) {
    u32x2_t r = {pack2(x[0], x[1]), pack2(x[2], x[3])};
    return __builtin_bit_cast(v4, r);
  }
};

struct F16Elem {
  static constexpr bool kFloatRange = false;
  typedef f16x8_t v8;
  typedef f16x4_t v4;
  static __device__ __forceinline__ float lo(uint32_t w) {
    return static_cast<float>(__builtin_bit_cast(f16x2_t, w)[0]);
  }
  static __device__ __forceinline__ float hi(uint32_t w) {
    return static_cast<float>(__builtin_bit_cast(f16x2_t, w)[1]);
  }
  static __device__ __forceinline__ uint32_t pack2(float a, float b) {  // round to nearest even
    f16x2_t v;
    v[0] = static_cast<_Float16>(a);
    v[1] = static_cast<_Float16>(b);
    return __builtin_bit_cast(uint32_t, v);
  }
  static __device__ __forceinline__ f32x16_t mfma32(v8 a, v8 b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ f32x4_t mfma16(v8 a, v8 b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ v4 read_tr(const unsigned char* p) {
    typedef __fp16 raw4 __attribute__((ext_vector_type(4)));
    typedef raw4 __attribute__((address_space(3))) * lds_v4;
    return __builtin_bit_cast(v4, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_v4)(p)));
  }
  static __device__ __forceinline__ f32x4_t mfma_k16(v4 a, v4 b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ v4 pack4(f32x4_t x) {
    u32x2_t r = {pack2(x[0], x[1]), pack2(x[2], x[3])};
    return __builtin_bit_cast(v4, r);
  }
};

template <class E>
struct Half64 {
  typedef E Elem;
  static constexpr int kMap = 0;  // what is done to the rows of Q and K: see FeatureMap
  typedef typename E::v8 v8_t;
  typedef typename E::v4 v4_t;
  static constexpr int D = 64, EPL = 8, NT = 4, kElemBytes = 2;
  static constexpr bool kFloatRange = E::kFloatRange, kPieces = false;
  // tiles in flight ahead of the one being processed, per pass (register budget permitting)
  static constexpr int kDepthState = 3, kDepthFwd = 3, kDepthQ = 2, kDepthKV = 2, kDepthQAccum = 1;
  // keep-all-tiles-in-registers variants of the fused kernels: forward only (the backward
  // does not have the registers)
  static constexpr bool kShortFwd = true, kShortBwd = false;
  static constexpr int kTileStride = mfma::kTileStride, kTileBytes = mfma::kTileBytes;
  static constexpr int kImageStride = 72;                 // elements per image row
  static constexpr int kImageBytes = D * kImageStride * 2;
  // Apply products leave lane (i16, g16) with the columns 32j + 8*g16 .. +7 (j = 0, 1) of tile
  // row i16: value 4*nt + v of the lane is column out_col(nt, g16) + v.  Image row n (an
  // output column of the product) is therefore kept at position image_row(n), which puts the
  // 16 rows one MFMA operand needs next to each other.
  static __device__ __forceinline__ int out_col(int nt, int g16) {
    return 32 * (nt >> 1) + 8 * g16 + 4 * (nt & 1);
  }
  static __device__ __forceinline__ int image_row(int n) {
    return 16 * (2 * (n >> 5) + ((n >> 2) & 1)) + 4 * ((n >> 3) & 3) + (n & 3);
  }

  // Products over 32 rows (32x32x16, W^T X^T as well) leave lane (row lane%32, half lane/32) with the columns
  // 32 nb + 16 t + 8 half .. + 7 (t = 0, 1: values 8 t .. of block nb), which is also what it holds of X: 16 bytes of
  // every 32.  Their images keep row n at rows32(n).
  struct Image32 {
    static __device__ __forceinline__ int rows32(int n) { return (n & ~12) | ((n & 4) << 1) | ((n & 8) >> 1); }
    static __device__ __forceinline__ int image_offset(int n, int k) { return (rows32(n) * kImageStride + k) * 2; }
  };
  // operand of columns 32 nb .. + 31 and the k of step ks (16 each)
  static __device__ __forceinline__ v8_t operand32(const unsigned char* image, int nb, int ks, const Lane& L) {
    return *reinterpret_cast<const v8_t*>(image + ((32 * nb + (L.lane & 31)) * kImageStride + 16 * ks + 8 * (L.lane >> 5)) * 2);
  }

  static __device__ __forceinline__ void unpack(const u32x4_t r, float (&f)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = E::lo(r[i]);
      f[2 * i + 1] = E::hi(r[i]);
    }
  }
  static __device__ __forceinline__ u32x4_t pack(const float (&f)[8]) {
    u32x4_t r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = E::pack2(f[2 * i], f[2 * i + 1]);
    return r;
  }

  static __device__ __forceinline__ float largest_raw(u32x4_t, float = 0.0f) { return 0.0f; }  // (no need to look)
  // the lane's EPL values (load layout: columns 8*ch ..) of tile row `row`
  template <bool = false>
  static __device__ __forceinline__ void put(unsigned char* T, int row, int ch, const float (&f)[8]) {
    put_raw(T, row, ch, pack(f));
  }
  template <bool = false>
  static __device__ __forceinline__ void put_raw(unsigned char* T, int row, int ch, u32x4_t r) {
    *reinterpret_cast<u32x4_t*>(T + row * kTileStride + ch * 16) = r;
  }

  // Operand of the 32x32x16 MFMA for a contraction over the 16 tile rows: lane gets, for
  // column cbase + lane%32, the 8 rows 8*(lane/32) .. +7 (two transposing reads of 4 rows).
  static __device__ __forceinline__ v8_t rows_operand(const unsigned char* T, const Lane& L,
                                                          int cbase) {
    const int s = L.i16;
    const int row = 8 * (L.g16 >> 1) + (s >> 2);
    const int col = cbase + 16 * (L.g16 & 1) + 4 * (s & 3);
    const unsigned char* p = T + row * kTileStride + col * 2;
    const v4_t lo = E::read_tr(p);
    const v4_t hi = E::read_tr(p + 4 * kTileStride);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }

  struct Acc {
    f32x16_t v[2][2];  // [row block of 32][column block of 32]
    __device__ __forceinline__ void zero() {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int i = 0; i < 16; ++i) v[a][c][i] = 0.0f;
    }
    // += (X tile)^T (Y tile)
    __device__ __forceinline__ void mfma(const unsigned char* Xt, const unsigned char* Yt,
                                         const Lane& L) {
      v8_t a[2], b[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        a[t] = rows_operand(Xt, L, 32 * t);
        b[t] = rows_operand(Yt, L, 32 * t);
      }
#pragma unroll
      for (int at = 0; at < 2; ++at)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
          v[at][ct] = E::mfma32(a[at], b[ct], v[at][ct]);
    }
    // group g = 0..15 of four consecutive state rows held by this lane, and where it lives
    __device__ __forceinline__ f32x4_t group(int g) const { return quad(v[g >> 3][(g >> 2) & 1], g & 3); }
    static __device__ __forceinline__ int group_row(int g, const Lane& L) {
      return 32 * (g >> 3) + 8 * (g & 3) + 4 * (L.lane >> 5);
    }
    static __device__ __forceinline__ int group_col(int g, const Lane& L) {
      return 32 * ((g >> 2) & 1) + (L.lane & 31);
    }
    static constexpr int kGroups = 16;
  };

  struct Operand {
    v8_t frag[4][2];
    __device__ __forceinline__ void load(const unsigned char* image, const Lane& L) {
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
          frag[nt][ks] = *reinterpret_cast<const v8_t*>(
              image + ((16 * nt + L.i16) * kImageStride + 8 * L.g16 + 32 * ks) * 2);
    }
  };

  // The 16 rows of an LDS tile as the other operand of an apply product: lane (i16, g16)
  // holds bytes 64j + 16*g16 .. +15 (j = 0, 1) of row i16, the same columns an apply product
  // leaves it with, so a tile fetched this way also serves as the epilogue's row operand.
  struct TileRows {
    v8_t a[2];
    __device__ __forceinline__ void load(const unsigned char* T, const Lane& L) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        a[ks] = *reinterpret_cast<const v8_t*>(T + L.i16 * kTileStride + (8 * L.g16 + 32 * ks) * 2);
    }
    // the two 16-byte pieces of the lane's row as 128-bit loads of global memory bring them
    template <bool = false>
    __device__ __forceinline__ void set(u32x4_t r0, u32x4_t r1) {
      a[0] = __builtin_bit_cast(v8_t, r0);
      a[1] = __builtin_bit_cast(v8_t, r1);
    }
    // from the row's values: f[8j + i] is column 32j + 8*g16 + i
    template <bool = false>
    __device__ __forceinline__ void set(const float (&f)[16]) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        float h[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) h[i] = f[8 * ks + i];
        a[ks] = __builtin_bit_cast(v8_t, Half64::pack(h));
      }
    }
    __device__ __forceinline__ void unpack(float (&f)[16]) const {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        float h[8];
        Half64::unpack(__builtin_bit_cast(u32x4_t, a[ks]), h);
#pragma unroll
        for (int i = 0; i < 8; ++i) f[8 * ks + i] = h[i];
      }
    }
    // Makes the next unpack() a fresh computation, so that the 16 floats of the previous
    // one need not stay in registers in between.
    __device__ __forceinline__ void forget_unpacked() {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        u32x4_t r = __builtin_bit_cast(u32x4_t, a[ks]);
        asm volatile("" : "+v"(r));
        a[ks] = __builtin_bit_cast(v8_t, r);
      }
    }
  };
  // (tile rows) x W, computed transposed (W^T X^T) so that each lane ends up with runs of
  // neighbouring columns of one row: out[nt][v] = T[row i16][column out_col(nt, g16) + v]
  static __device__ __forceinline__ void apply(const TileRows& X, const Operand& W,
                                               f32x4_t (&out)[4]) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      out[nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        out[nt] = E::mfma16(W.frag[nt][ks], X.a[ks], out[nt]);
    }
  }
  static __device__ __forceinline__ void apply(const unsigned char* T, const Operand& W,
                                               const Lane& L, f32x4_t (&out)[4]) {
    TileRows X;
    X.load(T, L);
    apply(X, W, out);
  }
  // out += (tile rows) x W
  static __device__ __forceinline__ void apply_onto(const TileRows& X, const Operand& W,
                                                    f32x4_t (&out)[4]) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) out[nt] = E::mfma16(W.frag[nt][ks], X.a[ks], out[nt]);
  }

  // columns nt of such a product, the operand fetched on the way (8 registers of it instead of 32)
  static __device__ __forceinline__ f32x4_t apply_columns(const TileRows& X, const unsigned char* image, int nt,
                                                          const Lane& L, f32x4_t d) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      d = E::mfma16(*reinterpret_cast<const v8_t*>(image + ((16 * nt + L.i16) * kImageStride + 8 * L.g16 + 32 * ks) * 2),
                    X.a[ks], d);
    return d;
  }

  // Products of two 16-row tiles, for the kernels that work tile pair by tile pair:
  // dots(a, b) = X_a X_b^T: lane (j, g) gets rows 4g .. 4g+3 (rows of a) of column j (row of b).
  static __device__ __forceinline__ f32x4_t dots(const TileRows& a, const TileRows& b,
                                                 f32x4_t d = f32x4_t{0.f, 0.f, 0.f, 0.f}) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) d = E::mfma16(a.a[ks], b.a[ks], d);
    return d;
  }
  // out += X^T P for the tile X at `T` and a 16 x 16 matrix P as dots() leaves it (rounded to
  // the element type): a 16x16 result leaves a lane with exactly the k it holds of a 16x16x16 B
  // operand, so P goes in without moving between lanes; X^T comes from the transposing LDS
  // read (lane i of a 16-lane group gets rows 4g .. 4g+3 of column out_col(nt, i/4) + i%4), so
  // the result lands in the product layout.
  typedef v4_t Weights;
  template <bool = false>
  static __device__ __forceinline__ Weights weights(f32x4_t p) {
    return E::pack4(p);
  }
  static __device__ __forceinline__ void add_transposed_product(const unsigned char* T,
                                                                const Lane& L, const Weights& p,
                                                                f32x4_t (&out)[4]) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
      out[nt] = E::mfma_k16(E::read_tr(T + (4 * L.g16 + (L.i16 >> 2)) * kTileStride +
                                       out_col(nt, L.i16 & 3) * 2),
                            p, out[nt]);
  }

  // One 32x32 block of a state, accumulated by one wave over LDS-resident tiles
  // (block = 0..3: rows 32*(block/2).., columns 32*(block%2)..), and its way into operand images.
  struct BlockAcc {
    static constexpr int kBlocks = 4;
    f32x16_t v;
    __device__ __forceinline__ void zero() {
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = 0.0f;
    }
    struct Frag {
      v8_t a, b;
    };
    static __device__ __forceinline__ Frag fetch(const unsigned char* Xt, const unsigned char* Yt,
                                                 const Lane& L, int block) {
      Frag f;
      f.a = rows_operand(Xt, L, 32 * (block >> 1));
      f.b = rows_operand(Yt, L, 32 * (block & 1));
      return f;
    }
    __device__ __forceinline__ void mma(const Frag& f) {
      v = E::mfma32(f.a, f.b, v);
    }
    // += (Y block)^T (X block): the transpose of what mma() adds
    __device__ __forceinline__ void mma_swapped(const Frag& f) {
      v = E::mfma32(f.b, f.a, v);
    }
    static __device__ __forceinline__ int run_row(int j, const Lane& L) { return 8 * j + 4 * (L.lane >> 5); }
    static __device__ __forceinline__ int run_col(const Lane& L) { return L.lane & 31; }
    // The lane holds, of the accumulated block, column lane%32 and rows 8j + 4*(lane/32) .. +3:
    // four neighbours of image row (c0 + column), which go out as one 64-bit write.
    //   after mma():          r0 = 32*(block/2), c0 = 32*(block%2)  ->  image[n][m] (transposed)
    //   after mma_swapped():  r0 = 32*(block%2), c0 = 32*(block/2)  ->  image[m][n] (natural)
    __device__ __forceinline__ void write_image(const Lane& L, int r0, int c0, float scale,
                                                unsigned char* image) const {
      const int c = c0 + (L.lane & 31);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = r0 + 8 * j + 4 * (L.lane >> 5);
        uint32_t* p = reinterpret_cast<uint32_t*>(image + (image_row(c) * kImageStride + r) * 2);
        p[0] = E::pack2(v[4 * j] * scale, v[4 * j + 1] * scale);
        p[1] = E::pack2(v[4 * j + 2] * scale, v[4 * j + 3] * scale);
      }
    }
    // Sum over this lane's elements of (accumulated block) x (the block of another matrix
    // read back from an image written by write_image with the same r0, c0).
    __device__ __forceinline__ float dot_image(const Lane& L, int r0, int c0,
                                               const unsigned char* image) const {
      const int c = c0 + (L.lane & 31);
      float s = 0.0f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = r0 + 8 * j + 4 * (L.lane >> 5);
        const uint32_t* p =
            reinterpret_cast<const uint32_t*>(image + (image_row(c) * kImageStride + r) * 2);
        const uint32_t lo = p[0], hi = p[1];
        s += v[4 * j] * E::lo(lo) + v[4 * j + 1] * E::hi(lo);
        s += v[4 * j + 2] * E::lo(hi) + v[4 * j + 3] * E::hi(hi);
      }
      return s;
    }
    static __device__ __forceinline__ int block_row0(int block) { return 32 * (block >> 1); }
    static __device__ __forceinline__ int block_col0(int block) { return 32 * (block & 1); }
  };

  // two neighbouring image elements (k, k+1) of image row n
  template <bool = false>
  static __device__ __forceinline__ void write_image_pair(unsigned char* image, int n, int k,
                                                          float v0, float v1) {
    *reinterpret_cast<uint32_t*>(image + (image_row(n) * kImageStride + k) * 2) = E::pack2(v0, v1);
  }
  // The same in two steps, for writers that split (n, k) into a per-lane and a compile-time part:
  // image_offset is additive over parts that share no bit of n (a permutation of bits) and in k.
  static __device__ __forceinline__ int image_offset(int n, int k) {
    return (image_row(n) * kImageStride + k) * 2;
  }
  template <bool = false>
  static __device__ __forceinline__ void write_four_at(unsigned char* at, f32x4_t v) {
    *reinterpret_cast<u32x2_t*>(at) = u32x2_t{E::pack2(v[0], v[1]), E::pack2(v[2], v[3])};
  }
  template <bool = false>
  static __device__ __forceinline__ void write_pair_at(unsigned char* at, float v0, float v1) {
    *reinterpret_cast<uint32_t*>(at) = E::pack2(v0, v1);
  }
  // what rounding the pair to the element type leaves off
  static __device__ __forceinline__ void left_over(float& v0, float& v1) {
    const uint32_t w = E::pack2(v0, v1);
    v0 -= E::lo(w);
    v1 -= E::hi(w);
  }
  // element k of image row n
  static __device__ __forceinline__ float image_at(const unsigned char* image, int n, int k) {
    const uint32_t h =
        *reinterpret_cast<const uint16_t*>(image + (image_row(n) * kImageStride + k) * 2);
    return E::lo(h);
  }
};

typedef Half64<Bf16Elem> Bf16x64;
typedef Half64<F16Elem> F16x64;

// fp32 rows on the bf16 matrix cores (1/16 of whose rate the fp32 products run at): a value is cut
// into three bf16 pieces, x = h + m + l exactly (8 + 8 + 8 of its 24 significant bits: h the
// upper half of the word, m the remainder rounded to bf16, l what is left, which fits), and a
// product of two values is the sum of the six products of pieces that reach its 24 bits,
//     h h' + (h m' + m h') + (h l' + l h' + m m'),
// each exact, accumulated in fp32.  What is left out (m l', l m', l l') is below 2^-22 of the product (m below
// 2^-7 of its value, l below 2^-16) and of either sign.  Six products at 16 times the rate: 2.7 times the fp32 matrix rate, for 11
// vector operations per pair of values cut.  Measured (a training step, us, fp32 products before and
// this): 512 slices x 200 rows, d_h = 128 333 and 202 (with the kernels of cotten_wide32.hip), d_h = 32
// 31.3 and 30.1; distance from a 64-bit evaluation 1.5e-7 ... 2.5e-7 and 1.1e-7 ... 1.5e-7.
//
// An infinity has no such pieces.  Its own are h = +-1, m = 0, l = +-inf: of the six products with a finite
// y, l h' is the infinity of the right sign (NaN for y = 0) and the others are finite, and of those
// with another infinity h l' and l h' are infinities of the same sign.  Rows that the cosine map divides by
// their length need no such care (an infinity makes them NaN); the others are looked over for one
// (one operation per pair of values) and cut again if there is one: write_pieces().
struct Pieces {
  bf16x8_t h, m, l;  // of eight values
};
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
  h = __builtin_amdgcn_perm(ub, ua, 0x07060302);  // the upper halves
  const float ra = a - __uint_as_float(ua & 0xffff0000u), rb = b - __uint_as_float(ub & 0xffff0000u);
  m = pack_bf16(ra, rb);
  asm("" : "+v"(m));  // (otherwise one of the pair is converted a second time for the next line)
  const float sa = ra - Bf16Elem::lo(m), sb = rb - Bf16Elem::hi(m);
  l = __builtin_amdgcn_perm(__float_as_uint(sb), __float_as_uint(sa), 0x07060302);
}
// n values, value i in half i % 2 of word i / 2.  INF: some may be infinite.
template <bool INF, int N>
__device__ __forceinline__ void split(const float (&v)[N], uint32_t (&h)[N / 2], uint32_t (&m)[N / 2],
                                      uint32_t (&l)[N / 2]) {
#pragma unroll
  for (int i = 0; i < N / 2; ++i) {
    split_pair(v[2 * i], v[2 * i + 1], h[i], m[i], l[i]);
    if (INF) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint32_t half = 0xffffu << (16 * j), word = __float_as_uint(v[2 * i + j]), sign = word & 0x80000000u;
        if ((word & 0x7fffffffu) != 0x7f800000u) continue;
        h[i] = (h[i] & ~half) | (sign | 0x3f800000u) >> (16 - 16 * j);
        m[i] &= ~half;
        l[i] = (l[i] & ~half) | word >> (16 - 16 * j);
      }
    }
  }
}
template <int N>
__device__ __forceinline__ float largest(const float (&v)[N], float so_far = 0.0f) {
#pragma unroll
  for (int i = 0; i < N; ++i) so_far = fmaxf(so_far, fabsf(v[i]));  // (NaN is passed over)
  return so_far;
}
__device__ __forceinline__ float largest(f32x4_t v, float so_far = 0.0f) {
  const float f[4] = {v[0], v[1], v[2], v[3]};
  return largest(f, so_far);
}
// write(std::false_type): values to where a product reads them, infinities not thought of; write(std::true_type), which
// is rarely run, if a lane of the wave has one (`largest`: the largest magnitude among the lane's values that may
// be infinite).  Decided ahead of the write and not behind it, so that nothing is kept for a second time.
template <class F, class Write>
__device__ __forceinline__ void write_pieces(float largest, Write&& write) {
  if constexpr (F::kPieces) {
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(largest == __builtin_inff()) != 0, 0)) write(std::true_type{});
    else write(std::false_type{});
  } else {
    write(std::false_type{});
  }
}
// the two values back, exactly
__device__ __forceinline__ float whole_lo(uint32_t h, uint32_t m, uint32_t l) {
  return Bf16Elem::lo(h) + (Bf16Elem::lo(m) + Bf16Elem::lo(l));
}
__device__ __forceinline__ float whole_hi(uint32_t h, uint32_t m, uint32_t l) {
  return Bf16Elem::hi(h) + (Bf16Elem::hi(m) + Bf16Elem::hi(l));
}

struct F32x32 {
  typedef float io_t;
  static constexpr bool kApart = false;
  static constexpr int kMap = 0;
  static constexpr int D = 32, EPL = 4, NT = 2, kElemBytes = 4;
  static constexpr bool kFloatRange = true, kPieces = true;
  static constexpr int kDepthState = 3, kDepthFwd = 3, kDepthQ = 3, kDepthKV = 2, kDepthQAccum = 2;
  static constexpr bool kShortFwd = true, kShortBwd = true;
  // A row of an LDS tile, or of an operand image: its 32 h pieces, its 32 m pieces, its 32 l pieces
  // (16 bytes of padding make the stride an odd number of 16-byte units).  Within a plane column
  // 16j + 4g + i sits at place 8g + 4j + i: the eight columns that a lane of group g holds in the
  // product layout next to each other.
  static constexpr int kPlane = 64, kTileStride = 3 * kPlane + 16, kTileBytes = TR * kTileStride;
  static constexpr int kImageStride = kTileStride;
  static constexpr int kImageBytes = D * kImageStride;
  static __device__ __forceinline__ int place(int column) {
    return 8 * ((column >> 2) & 3) + 4 * (column >> 4) + (column & 3);
  }
  static __device__ __forceinline__ int column(int place) {
    return 16 * ((place >> 2) & 1) + 4 * (place >> 3) + (place & 3);
  }
  // Apply products leave lane (i16, g16) with the columns 16j + 4*g16 .. +3 (j = 0, 1) of tile
  // row i16 (value 4*nt + v is column out_col(nt, g16) + v); image rows stay in place.
  static __device__ __forceinline__ int out_col(int nt, int g16) { return 16 * nt + 4 * g16; }

  static __device__ __forceinline__ void unpack(const u32x4_t r, float (&f)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(r[i]);
  }
  static __device__ __forceinline__ u32x4_t pack(const float (&f)[4]) {
    u32x4_t r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __float_as_uint(f[i]);
    return r;
  }

  static __device__ __forceinline__ float largest_raw(u32x4_t r, float so_far = 0.0f) {
    float f[4];
    unpack(r, f);
    return largest(f, so_far);
  }
  // four neighbouring places (multiples of four) of a plane row
  template <bool INF>
  static __device__ __forceinline__ void write_four(unsigned char* at, const float (&f)[4]) {
    uint32_t h[2], m[2], l[2];
    split<INF>(f, h, m, l);
    *reinterpret_cast<u32x2_t*>(at) = u32x2_t{h[0], h[1]};
    *reinterpret_cast<u32x2_t*>(at + kPlane) = u32x2_t{m[0], m[1]};
    *reinterpret_cast<u32x2_t*>(at + 2 * kPlane) = u32x2_t{l[0], l[1]};
  }
  // the lane's EPL values (load layout: columns 4*ch ..) of tile row `row`
  template <bool INF = false>
  static __device__ __forceinline__ void put(unsigned char* T, int row, int ch, const float (&f)[4]) {
    write_four<INF>(T + row * kTileStride + 16 * (ch & 3) + 8 * (ch >> 2), f);
  }
  template <bool INF = false>
  static __device__ __forceinline__ void put_raw(unsigned char* T, int row, int ch, u32x4_t r) {
    float f[4];
    unpack(r, f);
    put<INF>(T, row, ch, f);
  }

  static __device__ __forceinline__ f32x16_t mfma32(const Pieces& a, const Pieces& b, f32x16_t v) {
    v = Bf16Elem::mfma32(a.l, b.h, v);
    v = Bf16Elem::mfma32(a.h, b.l, v);
    v = Bf16Elem::mfma32(a.m, b.m, v);
    v = Bf16Elem::mfma32(a.m, b.h, v);
    v = Bf16Elem::mfma32(a.h, b.m, v);
    return Bf16Elem::mfma32(a.h, b.h, v);
  }
  // The same in two steps: all but the largest of the six products, and that one.  A sum over many tiles that takes the
  // small ones by themselves is rounded once per tile at its own size instead of six times.  (A tile's products from zero,
  // then added: the matrix instruction rounds off more beside a small addend, dK 1 x 16000 x 128 3.5e-7 against 1.9e-7.)
  static __device__ __forceinline__ f32x16_t mfma32_small(const Pieces& a, const Pieces& b, f32x16_t v) {
    v = Bf16Elem::mfma32(a.l, b.h, v);
    v = Bf16Elem::mfma32(a.h, b.l, v);
    v = Bf16Elem::mfma32(a.m, b.m, v);
    v = Bf16Elem::mfma32(a.m, b.h, v);
    return Bf16Elem::mfma32(a.h, b.m, v);
  }
  static __device__ __forceinline__ f32x16_t mfma32_large(const Pieces& a, const Pieces& b, f32x16_t v) {
    return Bf16Elem::mfma32(a.h, b.h, v);
  }
  static __device__ __forceinline__ f32x4_t mfma16(const Pieces& a, const Pieces& b, f32x4_t v) {
    v = Bf16Elem::mfma16(a.l, b.h, v);
    v = Bf16Elem::mfma16(a.h, b.l, v);
    v = Bf16Elem::mfma16(a.m, b.m, v);
    v = Bf16Elem::mfma16(a.m, b.h, v);
    v = Bf16Elem::mfma16(a.h, b.m, v);
    return Bf16Elem::mfma16(a.h, b.h, v);
  }
  // Operand of the 32x32x16 MFMA for a contraction over the 16 tile rows (see Half64): lane gets,
  // for place lane%32, the 8 rows 8*(lane/32) .. +7.
  static __device__ __forceinline__ bf16x8_t plane_operand(const unsigned char* p) {
    const bf16x4_t lo = Bf16Elem::read_tr(p);
    const bf16x4_t hi = Bf16Elem::read_tr(p + 4 * kTileStride);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }
  static __device__ __forceinline__ Pieces rows_operand(const unsigned char* T, const Lane& L) {
    const int row = 8 * (L.g16 >> 1) + (L.i16 >> 2), at = 16 * (L.g16 & 1) + 4 * (L.i16 & 3);
    const unsigned char* p = T + row * kTileStride + at * 2;
    return Pieces{plane_operand(p), plane_operand(p + kPlane), plane_operand(p + 2 * kPlane)};
  }
  static __device__ __forceinline__ bf16x8_t both(bf16x4_t a, bf16x4_t b) {
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  }
  // what a lane holds of a 32 x 32 result: column column(lane%32), and rows 16*(lane/32) + 4g .. +3
  static __device__ __forceinline__ int run_row(int g, const Lane& L) { return 4 * g + 16 * (L.lane >> 5); }
  static __device__ __forceinline__ int run_col(const Lane& L) { return column(L.lane & 31); }

  struct Acc {
    f32x16_t v;
    __device__ __forceinline__ void zero() {
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = 0.0f;
    }
    // += (X tile)^T (Y tile)
    __device__ __forceinline__ void mfma(const unsigned char* Xt, const unsigned char* Yt,
                                         const Lane& L) {
      add(rows_operand(Xt, L), rows_operand(Yt, L));
    }
    __device__ __forceinline__ void add(const Pieces& a, const Pieces& b) { v = mfma32(a, b, v); }
    __device__ __forceinline__ void add_lean(const Pieces& a, const Pieces& b) { v = mfma32(a, b, v); }
    __device__ __forceinline__ f32x4_t group(int g) const { return quad(v, g); }
    __device__ __forceinline__ void add_group(int g, f32x4_t x) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[4 * g + i] += x[i];
    }
    static __device__ __forceinline__ int group_row(int g, const Lane& L) { return run_row(g, L); }
    static __device__ __forceinline__ int group_col(int, const Lane& L) { return run_col(L); }
    static constexpr int kGroups = 4;
  };

  // frag[nt] = W[k][16*nt + i16] for the eight columns k that a TileRows lane holds.
  struct Operand {
    Pieces frag[2];
    __device__ __forceinline__ void load(const unsigned char* image, const Lane& L) {
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        const unsigned char* p = image + (16 * nt + L.i16) * kImageStride + 16 * L.g16;
        frag[nt].h = *reinterpret_cast<const bf16x8_t*>(p);
        frag[nt].m = *reinterpret_cast<const bf16x8_t*>(p + kPlane);
        frag[nt].l = *reinterpret_cast<const bf16x8_t*>(p + 2 * kPlane);
      }
    }
  };

  // Lane (i16, g16) holds bytes 64j + 16*g16 .. +15 (j = 0, 1) of tile row i16: the columns
  // an apply product leaves it with.
  struct TileRows {
    Pieces a;
    __device__ __forceinline__ void load(const unsigned char* T, const Lane& L) {
      const unsigned char* p = T + L.i16 * kTileStride + 16 * L.g16;
      a.h = *reinterpret_cast<const bf16x8_t*>(p);
      a.m = *reinterpret_cast<const bf16x8_t*>(p + kPlane);
      a.l = *reinterpret_cast<const bf16x8_t*>(p + 2 * kPlane);
    }
    // from the row's values: f[4j + i] is column 16j + 4*g16 + i
    template <bool INF = false>
    __device__ __forceinline__ void set(const float (&f)[8]) {
      uint32_t h[4], m[4], l[4];
      split<INF>(f, h, m, l);
      a = Pieces{__builtin_bit_cast(bf16x8_t, (u32x4_t{h[0], h[1], h[2], h[3]})),
                 __builtin_bit_cast(bf16x8_t, (u32x4_t{m[0], m[1], m[2], m[3]})),
                 __builtin_bit_cast(bf16x8_t, (u32x4_t{l[0], l[1], l[2], l[3]}))};
    }
    template <bool INF = false>
    __device__ __forceinline__ void set(u32x4_t r0, u32x4_t r1) {
      float f[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f[i] = __uint_as_float(r0[i]);
        f[4 + i] = __uint_as_float(r1[i]);
      }
      set<INF>(f);
    }
    __device__ __forceinline__ void unpack(float (&f)[8]) const {
      const u32x4_t h = __builtin_bit_cast(u32x4_t, a.h), m = __builtin_bit_cast(u32x4_t, a.m),
                    l = __builtin_bit_cast(u32x4_t, a.l);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f[2 * i] = whole_lo(h[i], m[i], l[i]);
        f[2 * i + 1] = whole_hi(h[i], m[i], l[i]);
      }
    }
    __device__ __forceinline__ void forget_unpacked() {}
  };
  static __device__ __forceinline__ void apply(const TileRows& X, const Operand& W,
                                               f32x4_t (&out)[2]) {
    out[0] = out[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    apply_onto(X, W, out);
  }
  static __device__ __forceinline__ void apply(const unsigned char* T, const Operand& W,
                                               const Lane& L, f32x4_t (&out)[2]) {
    TileRows X;
    X.load(T, L);
    apply(X, W, out);
  }
  // out += (tile rows) x W
  static __device__ __forceinline__ void apply_onto(const TileRows& X, const Operand& W,
                                                    f32x4_t (&out)[2]) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) out[nt] = mfma16(W.frag[nt], X.a, out[nt]);
  }

  // Products of two 16-row tiles (see Half64): dots(a, b) = X_a X_b^T, lane (j, g) gets rows
  // 4g .. 4g+3 of column j.
  static __device__ __forceinline__ f32x4_t dots(const TileRows& a, const TileRows& b,
                                                 f32x4_t d = f32x4_t{0.f, 0.f, 0.f, 0.f}) {
    return mfma16(a.a, b.a, d);
  }
  // out += X^T P (see Half64).  The contraction runs over 16 rows where a 16x16x32 product takes 32:
  // the two halves of its depth carry two products of pieces at a time, three instead of six.
  // INF: P may hold infinities.
  struct Weights {
    bf16x8_t hh, mm, hl;
  };
  template <bool INF = false>
  static __device__ __forceinline__ Weights weights(f32x4_t p) {
    const float f[4] = {p[0], p[1], p[2], p[3]};
    uint32_t h[2], m[2], l[2];
    write_pieces<F32x32>(INF ? largest(f) : 0.0f, [&](auto inf) { split<decltype(inf)::value>(f, h, m, l); });
    const bf16x4_t bh = __builtin_bit_cast(bf16x4_t, (u32x2_t{h[0], h[1]})), bm = __builtin_bit_cast(bf16x4_t, (u32x2_t{m[0], m[1]})),
                   bl = __builtin_bit_cast(bf16x4_t, (u32x2_t{l[0], l[1]}));
    return Weights{both(bh, bh), both(bm, bm), both(bh, bl)};
  }
  static __device__ __forceinline__ void add_transposed_product(const unsigned char* T,
                                                                const Lane& L, const Weights& p,
                                                                f32x4_t (&out)[2]) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      const unsigned char* at =
          T + (4 * L.g16 + (L.i16 >> 2)) * kTileStride + (8 * (L.i16 & 3) + 4 * nt) * 2;
      const bf16x4_t xh = Bf16Elem::read_tr(at), xm = Bf16Elem::read_tr(at + kPlane),
                     xl = Bf16Elem::read_tr(at + 2 * kPlane);
      const bf16x8_t xhm = both(xh, xm);
      out[nt] = Bf16Elem::mfma16(both(xl, xh), p.hl, out[nt]);  // l h' + h l'
      out[nt] = Bf16Elem::mfma16(xhm, p.mm, out[nt]);           // h m' + m m'
      out[nt] = Bf16Elem::mfma16(xhm, p.hh, out[nt]);           // h h' + m h'
    }
  }
  // The state as the one 32 x 32 block it is (see Half64::BlockAcc).
  struct BlockAcc {
    static constexpr int kBlocks = 1;
    f32x16_t v;
    __device__ __forceinline__ void zero() {
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = 0.0f;
    }
    struct Frag {
      Pieces a, b;
    };
    static __device__ __forceinline__ Frag fetch(const unsigned char* Xt, const unsigned char* Yt,
                                                 const Lane& L, int) {
      return Frag{rows_operand(Xt, L), rows_operand(Yt, L)};
    }
    __device__ __forceinline__ void mma(const Frag& f) { v = mfma32(f.a, f.b, v); }
    __device__ __forceinline__ void mma_swapped(const Frag& f) { v = mfma32(f.b, f.a, v); }
    static __device__ __forceinline__ int run_row(int j, const Lane& L) { return F32x32::run_row(j, L); }
    static __device__ __forceinline__ int run_col(const Lane& L) { return F32x32::run_col(L); }
    __device__ __forceinline__ void write_image(const Lane& L, int r0, int c0, float scale,
                                                unsigned char* image) const {
      float top = 0.0f;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        top = largest(quad(v, j) * scale, top);
      write_pieces<F32x32>(top, [&](auto inf) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          write_four_at<decltype(inf)::value>(image + image_offset(c0 + run_col(L), r0 + run_row(j, L)), quad(v, j) * scale);
      });
    }
    static __device__ __forceinline__ int block_row0(int) { return 0; }
    static __device__ __forceinline__ int block_col0(int) { return 0; }
  };

  template <bool INF = false>
  static __device__ __forceinline__ void write_image_pair(unsigned char* image, int n, int k,
                                                          float v0, float v1) {
    write_pair_at<INF>(image + image_offset(n, k), v0, v1);
  }
  static __device__ __forceinline__ int image_offset(int n, int k) {
    return n * kImageStride + place(k) * 2;
  }
  template <bool INF = false>
  static __device__ __forceinline__ void write_four_at(unsigned char* at, f32x4_t v) {
    const float f[4] = {v[0], v[1], v[2], v[3]};
    write_four<INF>(at, f);
  }
  template <bool INF = false>
  static __device__ __forceinline__ void write_pair_at(unsigned char* at, float v0, float v1) {
    const float f[2] = {v0, v1};
    uint32_t h[1], m[1], l[1];
    split<INF>(f, h, m, l);
    *reinterpret_cast<uint32_t*>(at) = h[0];
    *reinterpret_cast<uint32_t*>(at + kPlane) = m[0];
    *reinterpret_cast<uint32_t*>(at + 2 * kPlane) = l[0];
  }
  static __device__ __forceinline__ float image_at(const unsigned char* image, int n, int k) {
    const uint16_t* p = reinterpret_cast<const uint16_t*>(image + image_offset(n, k));
    return whole_lo(p[0], p[kPlane / 2], p[kPlane]);
  }
};

// The same rows, with states whose small products are summed apart from the large one, for the sums that run over whole
// sequences or long parts of them (error of dK against float64, 64 slices x 3500 rows, d_h = 128: 3.7e-7 without, 2.1e-7
// with).  Where three or more workgroups share a compute unit the registers cost time (419 slices x 736 rows, d_h = 32,
// backward 71.1 us without, 72.7 with): those keep the plain format.
struct F32x32Apart : F32x32 {
  static constexpr bool kApart = true;
  // (one tile ahead while two states' worth of accumulators are live: three waves per SIMD instead of two, split
  // backward 90 slices x 2000 rows, d_h = 32, 48.3 -> 44.4 us)
  static constexpr int kDepthQAccum = 1;
  struct Acc : F32x32::Acc {
    f32x16_t small;  // the sum of the small products
    __device__ __forceinline__ void zero() {
      F32x32::Acc::zero();
#pragma unroll
      for (int i = 0; i < 16; ++i) small[i] = 0.0f;
    }
    __device__ __forceinline__ void mfma(const unsigned char* Xt, const unsigned char* Yt, const Lane& L) {
      add(rows_operand(Xt, L), rows_operand(Yt, L));
    }
    __device__ __forceinline__ void add(const Pieces& a, const Pieces& b) {
      small = mfma32_small(a, b, small);
      v = mfma32_large(a, b, v);
    }
    // without a second accumulator: the tile's small products first, by themselves
    __device__ __forceinline__ void add_lean(const Pieces& a, const Pieces& b) {
      f32x16_t t;
#pragma unroll
      for (int i = 0; i < 16; ++i) t[i] = 0.0f;
      t = mfma32_small(a, b, t);
      v = mfma32_large(a, b, v);
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] += t[i];
    }
    __device__ __forceinline__ f32x4_t group(int g) const { return quad(v, g) + quad(small, g); }
  };
};

// What a format does to the rows of Q and K before they enter the products:
//   kMapCosine  x / sqrt(|x|^2 + eps)   row-wise L2 normalisation (the paper's model)
//   kMapElu1    ELU(x) + 1              element-wise (the linear-attention comparison model of
//                                       "Linear Attention Models"); eps plays no part
// A format with the second map is the same format with kMap overridden: every pass picks the
// staging mode and the row epilogue from F::kMap.
enum FeatureMap { kMapCosine = 0, kMapElu1 = 1 };
template <class Base>
struct WithElu1 : Base {
  static constexpr int kMap = kMapElu1;
};

// phi(x) = ELU(x) + 1 with alpha = 1: x + 1 above zero, exp(x) below (hardware exp2, about
// 1 ulp).  Its derivative is 1 above zero and exp(x) below, i.e. min(phi(x), 1).
__device__ __forceinline__ float elu1(float x) {
  return x > 0.0f ? x + 1.0f : __builtin_amdgcn_exp2f(x * 1.44269504088896340736f);
}
// (selects: with the condition around the call a branch per value, bf16 256 slices x 400 rows forward 16.8 -> 19.2 us)
__device__ __forceinline__ float elu1_or_zero(float x, bool on) {
  const float below = __builtin_amdgcn_exp2f(x * 1.44269504088896340736f), above = x + 1.0f;
  const float phi = x > 0.0f ? above : below;
  return on ? phi : 0.0f;
}

// ---- tiles --------------------------------------------------------------------------------

// The tiles one workgroup walks: local tile lt = 0 .. n_tiles-1 is tile (tile0 + lt * stride)
// of the slice, i.e. rows 16*(tile0 + lt*stride) .. +15.  A fused workgroup has stride 1; in
// the split path the tiles of a slice are dealt round-robin to its `splits` workgroups, so
// that padding (which sits at one end of the sequence) is shared evenly.  Rows >= limit do
// not exist; `flags`, if given, is the LDS copy of the key mask: flags[16*lt + r].
struct Rows {
  int tile0, stride, n_tiles, limit;
  const uint8_t* flags;
  __device__ __forceinline__ int row0(int lt) const { return (tile0 + lt * stride) * TR; }
};

// Raw 16-row tile in the load layout: x[h], y[h] hold row r8 + 8h; `live` bit h says the
// row takes part (in range and, where a mask applies, a valid key).
struct Raw {
  u32x4_t x[2], y[2];
  int live;
};

// The two tensors a pass reads, as buffer resources over one slice each.  Buffer loads are
// used instead of flat loads because a lane whose offset lies outside the buffer gets zeros
// and causes no memory traffic: rows that do not take part are skipped without a branch, so
// every tile issues the same number of load instructions and the hardware's in-order load
// counter can tell "this tile has arrived" from "the tiles prefetched after it have not".
// How the rows of a slice are addressed in global memory: `stride` bytes apart, `bytes` bytes
// each (128, or 64 / 32 for narrower rows: d_h = 32 or 16 with 16-bit elements, d_h = 16 with
// fp32 - those run on the full-width formats with the rest of every tile row held at zero,
// which leaves all results unchanged).
struct RowAddr {
  int stride, bytes;
};

// Where the slices are (bytes): slice (b,h) starts at b*batch + h*head.
// [B,H,N,d]: batch = H*N*row bytes, head = N*row bytes, stride = row bytes;
// [B,N,H,d]: batch = N*H*row bytes, head = row bytes, stride = H*row bytes.
struct Strides {
  long long batch, head;
  RowAddr row;
  __device__ __forceinline__ size_t slice_base(int bh, int H) const {
    return static_cast<size_t>(bh / H) * batch + static_cast<size_t>(bh % H) * head;
  }
};

struct Src {
  __amdgpu_buffer_rsrc_t x, y;
  RowAddr row;
  __device__ __forceinline__ Src(const unsigned char* X, const unsigned char* Y, int N,
                                 RowAddr row_addr)
      : row(row_addr) {
    const int bytes = (N - 1) * row.stride + row.bytes;
    x = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(X), 0, bytes, 0x00020000);
    y = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(Y), 0, bytes, 0x00020000);
  }
  // byte offset of the lane's 16 bytes of `row`, outside the buffer (zeros, no traffic) when
  // the row does not take part or the lane's columns are padding
  __device__ __forceinline__ uint32_t offset(int row_index, bool live, const Lane& L) const;
};
constexpr uint32_t kOutOfBuffer = 0x80000000u;
__device__ __forceinline__ uint32_t Src::offset(int row_index, bool live, const Lane& L) const {
  return (live && L.ch * 16 < row.bytes) ? static_cast<uint32_t>(row_index) * row.stride + L.ch * 16
                                         : kOutOfBuffer;
}

// Loads local tile lt (all zeros, and no traffic, if lt is not one of the workgroup's tiles).
// A row takes part when it is below rows.limit and, if rows.flags is given, its flag is set.
template <bool USE_Y>
__device__ __forceinline__ void load_raw(Raw& r, const Lane& L, const Src& src, const Rows& rows,
                                         int lt) {
  r.live = 0;
  const bool tile_ok = lt < rows.n_tiles;
  const int row0 = rows.row0(lt);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = row0 + L.r8 + 8 * h;
    bool live = tile_ok && row < rows.limit;
    if (rows.flags != nullptr) live = live && rows.flags[tile_ok ? lt * TR + L.r8 + 8 * h : 0] != 0;
    const uint32_t off = src.offset(row, live, L);
    r.x[h] = __builtin_amdgcn_raw_buffer_load_b128(src.x, off, 0, 0);
    if (USE_Y) r.y[h] = __builtin_amdgcn_raw_buffer_load_b128(src.y, off, 0, 0);
    else r.y[h] = u32x4_t{0, 0, 0, 0};
    r.live |= static_cast<int>(live) << h;
  }
}

// What becomes of the x rows on their way to the LDS tile.
enum XMode { kXNone = 0, kXRaw = 1, kXNormalized = 2, kXFeature = 3 };

// The staging mode of rows that enter a product through the feature map of the format.
template <class F>
constexpr int mapped_mode() {
  return F::kMap == kMapElu1 ? kXFeature : kXNormalized;
}

// inv[h] = 1/r of row h (0, with MARK -0, for rows that do not take part; their registers are zero).
// Xt receives nothing, the raw rows, xhat, or phi(x) (kXFeature: then inv[h] is 1 for a row
// that takes part, and `cols` says whether the lane's columns exist - phi(0) is not 0, so
// padding columns and absent rows are written as zeros explicitly); Yt the raw y rows.
template <class F, int XMODE, bool USE_Y, bool MARK = false>
__device__ __forceinline__ void stage(const Raw& r, const Lane& L, float eps, unsigned char* Xt,
                                      unsigned char* Yt, float (&inv)[2], bool cols = true) {
  // one row: x (INF: phi(x) may be infinite), y
  const auto stage_x = [&](int h, auto inf) {
    float f[F::EPL];
    F::unpack(r.x[h], f);
    const int row = L.r8 + 8 * h;
    if (XMODE == kXFeature) {
      const bool live = ((r.live >> h) & 1) != 0, on = live & cols;
      inv[h] = live ? 1.0f : MARK ? -0.0f : 0.0f;
#pragma unroll
      for (int i = 0; i < F::EPL; ++i) f[i] = elu1_or_zero(f[i], on);
      F::template put<decltype(inf)::value>(Xt, row, L.ch, f);
      return;
    }
    float ss = 0.0f;
#pragma unroll
    for (int i = 0; i < F::EPL; ++i) ss += f[i] * f[i];
    inv[h] = inv_norm_or_zero<MARK>(row_sum8(ss), eps, (r.live >> h) & 1);
    if (XMODE == kXNormalized) {
#pragma unroll
      for (int i = 0; i < F::EPL; ++i) f[i] *= inv[h];
      F::put(Xt, row, L.ch, f);
    } else if (XMODE == kXRaw) {
      F::put_raw(Xt, row, L.ch, r.x[h]);
    }
  };
  const auto stage_y = [&](int h, auto inf) {
    if (USE_Y) F::template put_raw<decltype(inf)::value>(Yt, L.r8 + 8 * h, L.ch, r.y[h]);
  };
  if constexpr (!F::kPieces) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      stage_x(h, std::false_type{});
      stage_y(h, std::false_type{});
    }
    return;
  }
  // (y is looked at behind x: it may still be on its way)
  write_pieces<F>(XMODE == kXFeature ? F::largest_raw(r.x[0], F::largest_raw(r.x[1])) : 0.0f, [&](auto inf) {
    stage_x(0, inf);
    stage_x(1, inf);
  });
  write_pieces<F>(USE_Y ? F::largest_raw(r.y[0], F::largest_raw(r.y[1])) : 0.0f, [&](auto inf) {
    stage_y(0, inf);
    stage_y(1, inf);
  });
}

// ---- epilogues in the product layout ------------------------------------------------------
// An apply product leaves lane (i16, g16) with 2*EPL values of tile row i16: the two 16-byte
// pieces of the row at bytes 64j + 16*g16.  TileRows::unpack gives any LDS tile in the same
// arrangement, so row-wise epilogues need no detour through an fp32 scratch tile.

template <class F>
__device__ __forceinline__ void product_rows(const f32x4_t (&out)[F::NT], float (&p)[2 * F::EPL]) {
  static_assert(4 * F::NT == 2 * F::EPL, "an apply product covers one row");
#pragma unroll
  for (int nt = 0; nt < F::NT; ++nt)
#pragma unroll
    for (int v = 0; v < 4; ++v) p[4 * nt + v] = out[nt][v];
}

// Sum over the 64 lanes of the wave, every lane gets it (fixed butterfly order).
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int w = 1; w < 64; w <<= 1) x += __shfl_xor(x, w);
  return x;
}

// Sum over the four lanes (i16, 0..3) that share a row.
__device__ __forceinline__ float row_sum_groups(float x, const Lane& L) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((L.lane ^ 16) << 2, __builtin_bit_cast(int, x)));
  x += __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((L.lane ^ 32) << 2, __builtin_bit_cast(int, x)));
  return x;
}

// p <- (p - u (u.p)) / r for the lane's row, u being the unit row held in `e`: the tangent
// projection shared by dQ (u = qhat, p = g) and dK (u = khat, p = h).  With LAZY the unit row
// is unpacked twice instead of being kept in registers across the row sum.
template <class F, bool LAZY>
__device__ __forceinline__ void project_rows(float (&p)[2 * F::EPL], typename F::TileRows& e,
                                             float inv_r, const Lane& L) {
  float u[2 * F::EPL];
  e.unpack(u);
  float proj = 0.0f;
#pragma unroll
  for (int c = 0; c < 2 * F::EPL; ++c) proj += u[c] * p[c];
  proj = row_sum_groups(proj, L);
  if (LAZY) {
    e.forget_unpacked();
    e.unpack(u);
  }
#pragma unroll
  for (int c = 0; c < 2 * F::EPL; ++c) p[c] = (p[c] - u[c] * proj) * inv_r;
}

// p <- p * phi'(x) element-wise, with phi(x) of the lane's row held in `e`: the chain rule
// through the ELU + 1 map (phi' = min(phi, 1)).
template <class F>
__device__ __forceinline__ void feature_grad_rows(float (&p)[2 * F::EPL],
                                                  const typename F::TileRows& e) {
  float u[2 * F::EPL];
  e.unpack(u);
#pragma unroll
  for (int c = 0; c < 2 * F::EPL; ++c) p[c] *= fminf(u[c], 1.0f);
}

// The same with the raw row x = r * u:  (p - u (u.p)) / r = (p - x (x.p) / r^2) / r.
template <class F>
__device__ __forceinline__ void project_values(float (&p)[2 * F::EPL], const float (&x)[2 * F::EPL],
                                               float inv_r, const Lane& L) {
  float proj = 0.0f;
#pragma unroll
  for (int c = 0; c < 2 * F::EPL; ++c) proj += x[c] * p[c];
  // one factor at a time: 1/r^2 alone leaves the fp32 range for rows next to zero, and (x.p) / r^3 for long ones
  proj = row_sum_groups(proj, L) * inv_r * inv_r;
#pragma unroll
  for (int c = 0; c < 2 * F::EPL; ++c) p[c] = (p[c] - x[c] * proj) * inv_r;
}
template <class F>
__device__ __forceinline__ void project_rows_raw(float (&p)[2 * F::EPL],
                                                 const typename F::TileRows& e, float inv_r,
                                                 const Lane& L) {
  float x[2 * F::EPL];
  e.unpack(x);
  project_values<F>(p, x, inv_r, L);
}

// Cache policy of the result stores.  Results are not read again by these kernels, and with
// the default policy the written lines displace the inputs still on their way through L2.
// Measured at N = 200 on the benchmark's alternating forward / backward steps (tokens/s of the
// step, fp32 fused and bf16 resident kernels): default 1.6 G and 0.77 G; nt 1.88 G and 0.90 G;
// sc0 sc1 nt 1.91 G and 0.93 G; sc0 sc1 without nt is the best for a forward run on its own
// but loses 8 % in the step.  The split kernels (N = 4096): default 0.64 G, nt 0.63 G, sc0 sc1
// 0.63 G, sc0 sc1 nt 0.67 G.  Loads are better left with the default policy everywhere.
constexpr int kStoreDefault = 0, kStoreStreamed = 19;  // aux bits: sc0 = 1, nt = 2, sc1 = 16

template <class F, int POLICY>
__device__ __forceinline__ void store_product_row(unsigned char* __restrict__ dst, int row,
                                                  RowAddr addr, const Lane& L,
                                                  const float (&p)[2 * F::EPL]) {
  // dst is a slice base: the byte offsets of its rows fit 31 bits (checked by the caller of
  // the library entry point)
  __amdgpu_buffer_rsrc_t out;
  if (POLICY != kStoreDefault) out = __builtin_amdgcn_make_buffer_rsrc(dst, 0, 0x7fffffff, 0x00020000);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (64 * j + 16 * L.g16 >= addr.bytes) break;  // narrower rows: the rest is padding
    float c[F::EPL];
#pragma unroll
    for (int i = 0; i < F::EPL; ++i) c[i] = p[F::EPL * j + i];
    const uint32_t off = static_cast<uint32_t>(row) * addr.stride + 64 * j + 16 * L.g16;
    if (POLICY != kStoreDefault) __builtin_amdgcn_raw_buffer_store_b128(F::pack(c), out, off, 0, POLICY);
    else *reinterpret_cast<u32x4_t*>(dst + off) = F::pack(c);
  }
}

// ---- rows that only their own wave reads ---------------------------------------------------

// The wave's own 16 rows of one tensor, loaded from global memory in the layout of the products
// (lane (i16, g16): bytes 128 c + 64 j + 16 g16 .. + 15 of row i16), so that they need no LDS at all.
template <int P>
struct OwnRaw {
  u32x4_t r[P][2];
};

struct Buffers {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ Buffers(const unsigned char* base, int N, RowAddr row) {
    r = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(base), 0,
                                          (N - 1) * row.stride + row.bytes, 0x00020000);
  }
};

template <int P>
__device__ __forceinline__ void load_own(OwnRaw<P>& t, const Lane& L, __amdgpu_buffer_rsrc_t X, RowAddr addr,
                                         int row0, bool live) {
  const uint32_t at = static_cast<uint32_t>(row0 + L.i16) * addr.stride + L.g16 * 16;
#pragma unroll
  for (int c = 0; c < P; ++c)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = c * kRowBytes + 64 * j;
      t.r[c][j] = __builtin_amdgcn_raw_buffer_load_b128(
          X, live && col + L.g16 * 16 < addr.bytes ? at + col : kOutOfBuffer, 0, 0);
    }
}
template <int P>
__device__ __forceinline__ void load_own(OwnRaw<P>& t, const Lane& L, const Buffers& X, RowAddr addr,
                                         int row0, bool live) {
  load_own<P>(t, L, X.r, addr, row0, live);
}

// The lane's values of piece c.
template <class F, int P>
__device__ __forceinline__ void own_values(const OwnRaw<P>& t, int c, float (&f)[2 * F::EPL]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    float h[F::EPL];
    F::unpack(t.r[c][j], h);
#pragma unroll
    for (int i = 0; i < F::EPL; ++i) f[F::EPL * j + i] = h[i];
  }
}

// (INF: rows that the cosine map does not divide by their length)
template <class F, int P, bool INF>
__device__ __forceinline__ void own_rows(const OwnRaw<P>& t, typename F::TileRows (&x)[P]) {
  float top = 0.0f;
  if (F::kPieces && INF) {
#pragma unroll
    for (int c = 0; c < P; ++c) {
      float f[2 * F::EPL];
      own_values<F, P>(t, c, f);
      top = largest(f, top);
    }
  }
  write_pieces<F>(top, [&](auto inf) {
#pragma unroll
    for (int c = 0; c < P; ++c) x[c].template set<decltype(inf)::value>(t.r[c][0], t.r[c][1]);
  });
}

// ---- states into operand images --------------------------------------------------------------

// A quadrant of scale * M from the accumulator layout (`get(g)`: group g, four consecutive rows of
// one column) into its operand image: transposed straight from the lane (two row pairs of its
// column), natural with the neighbouring lane's column (even lanes write the first two rows of a
// group, odd lanes the last two; each gets the other column of its rows from its neighbour).
// IMAGE: the order of the image's rows (F, or F::Image32).
template <class F, bool NATURAL, class IMAGE = F, class Get>
__device__ __forceinline__ void quadrant_image(Get get, float scale, unsigned char* image, const Lane& L) {
  // (row, column) of the first value of a group = a part that depends on the lane only plus a
  // part that depends on the group only; the image offsets of the two add up, so the second
  // becomes the immediate offset of the write
  const int lane_row = F::Acc::group_row(0, L), lane_col = F::Acc::group_col(0, L);
  const bool odd = (lane_col & 1) != 0;
  Lane zero = L;
  zero.set(0);
  unsigned char* at = image + (NATURAL ? IMAGE::image_offset(lane_row + (odd ? 2 : 0), lane_col & ~1)
                                       : IMAGE::image_offset(lane_col, lane_row));
  if constexpr (NATURAL && F::kElemBytes == 2) {
    // 16 bits: rounded first, so that one move per group brings the neighbour's column of both rows
    const uint32_t lows = odd ? 0x01000504u : 0x05040100u, highs = odd ? 0x03020706u : 0x07060302u;
#pragma unroll
    for (int g = 0; g < F::Acc::kGroups; ++g) {
      const f32x4_t v = get(g) * scale;
      const int row = F::Acc::group_row(g, zero), col = F::Acc::group_col(g, zero);
      const uint32_t first = F::Elem::pack2(v[0], v[1]), second = F::Elem::pack2(v[2], v[3]);
      const uint32_t mine = odd ? second : first;
      int sent = static_cast<int>(odd ? first : second);  // (chosen on the sending side, see below)
      asm volatile("" : "+v"(sent));
      int got = __builtin_amdgcn_update_dpp(0, sent, 0xB1, 0xF, 0xF, true);  // lane ^ 1
      asm volatile("" : "+v"(got));
      // (mine: bytes 0 ... 3 of the pair of words, got: 4 ... 7)
      *reinterpret_cast<uint32_t*>(at + IMAGE::image_offset(row, col)) = __builtin_amdgcn_perm(got, mine, lows);
      *reinterpret_cast<uint32_t*>(at + IMAGE::image_offset(row + 1, col)) = __builtin_amdgcn_perm(got, mine, highs);
    }
    return;
  }
  float top = 0.0f;
  if (F::kPieces) {
#pragma unroll
    for (int g = 0; g < F::Acc::kGroups; ++g) top = largest(get(g) * scale, top);
  }
  write_pieces<F>(top, [&](auto inf) {
    constexpr bool kInf = decltype(inf)::value;
#pragma unroll
    for (int g = 0; g < F::Acc::kGroups; ++g) {
      const f32x4_t v = get(g) * scale;
      const int row = F::Acc::group_row(g, zero), col = F::Acc::group_col(g, zero);  // the group's part
      if (!NATURAL) {
        F::template write_four_at<kInf>(at + IMAGE::image_offset(col, row), v);
      } else {
        // The lane sends what its neighbour wants (the choice is made on the sending side: a
        // choice between two values received from the neighbour would be evaluated over there).
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float mine = odd ? v[2 + i] : v[i];
          int sent = __builtin_bit_cast(int, odd ? v[i] : v[2 + i]);
          asm volatile("" : "+v"(sent));
          int got = __builtin_amdgcn_update_dpp(0, sent, 0xB1, 0xF, 0xF, true);  // lane ^ 1
          asm volatile("" : "+v"(got));
          const float other = __builtin_bit_cast(float, got);
          F::template write_pair_at<kInf>(at + IMAGE::image_offset(row + i, col), odd ? other : mine, odd ? mine : other);
        }
      }
    }
  });
}

}  // namespace mfma
}  // namespace cotten
