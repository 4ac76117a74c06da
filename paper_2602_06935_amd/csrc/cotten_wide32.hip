// fp32 rows of 256 and 512 bytes (d_h = 64 and 128) on the matrix cores: a row in P = 2 or 4 pieces of
// 128 bytes, a state in P x P blocks of 32 x 32, every product as six products of bf16 pieces
// (F32x32 in cotten_mfma_core.h).
//
//     S[p][q]  = sum_j khat_j[piece p]^T v_j[piece q]                     (state walk)
//     O[q]     = sum_p Qhat[piece p] S[p][q]       likewise dQ, dK, dV    (apply)
//
// State walk: the rows go through LDS, where the matrix cores read them transposed, cut into
// pieces once on the way.
//   P = 2  a workgroup of four waves; a wave adds its own tiles to a state of its own (no barriers),
//          the four sums meet at the end
//   P = 4  eight waves, rounds of 64 rows staged by all of them; a wave adds two of the four tiles of
//          a round to a quadrant of 2 x 2 blocks, the two sums of a quadrant meet at the end
// Apply: a wave loads its own rows straight in the layout of the products (no LDS), the state is
// read from the operand images.
//
// A sequence that is not cut takes one launch per direction and the state never leaves the compute
// unit; the backward has two roles, side by side on one XCD, each of which reads all four tensors:
//   S from (K, V), then dQ;      dS from (Q, dO), then dV and dK
// A cut one takes three launches: partial states into the caller's workspace, their sum in split
// order (reduce_states_kernel), apply (backward: dQ, dV, dK as three roles).
#include "cotten_launch.h"
#include "cotten_mfma_core.h"

namespace cotten {
namespace {
namespace wide32 {

using namespace mfma;

extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

template <int P>
constexpr int waves() { return P == 2 ? 4 : 8; }

// LDS: the tiles of the state walk; over them, once the state is complete, the sums that meet and
// then the operand images (P = 2: two sets, P = 4: one); behind them a few words.
template <class F, int P>
struct Lds {
  static constexpr int kPair = 2 * P * F::kTileBytes;   // [x pieces | y pieces] of 16 rows
  static constexpr int kTiles = 4 * kPair;              // P = 2: one pair per wave; P = 4: a round of 64 rows
  static constexpr int kSet = P * P * F::kImageBytes;
  static constexpr int kSets = P == 2 ? 2 : 1;
  static constexpr int kMeet = P == 2 ? 12 * 4096 : 16 * 4096;
  static constexpr int kWords = kTiles;
  static constexpr int kBytes = kWords + 64;
  static_assert(kSets * kSet <= kTiles && kMeet <= kTiles, "images and sums lie over the tiles");
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
  int H, N, slices;
  float scale, eps;
  const float* slice_scale;
  float* kept;             // forward: S of every slice, or nullptr
  float* dlog;             // backward: d loss / d log(scale) of every slice, or nullptr
  int splits, rows_per_split;
  const float* states;     // three launches: the complete states
  const float* dstates;
  Strides st;
  __device__ __forceinline__ float scale_of(int bh) const {
    return slice_scale != nullptr ? slice_scale[bh] : scale;
  }
  __device__ __forceinline__ const uint8_t* keys_of(int bh) const {
    return mask == nullptr ? nullptr : mask + static_cast<size_t>(bh / H) * N;
  }
};

// ---- state walk -------------------------------------------------------------------------------------

// 16 rows of one tensor in the load layout: r[h][c] is bytes 128 c + 16 ch .. + 15 of row r8 + 8 h.
template <int P>
struct Half16 {
  u32x4_t r[2][P];
};

__device__ __forceinline__ int row_bits(const uint8_t* __restrict__ mask, int row0, int end, const Lane& L) {
  int bits = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = row0 + L.r8 + 8 * h;
    if (row < end) bits |= static_cast<int>(mask == nullptr || mask[row] != 0) << h;
  }
  return bits;
}

template <int P>
__device__ __forceinline__ void load_half(Half16<P>& t, const Lane& L, const Buffers& X, int stride, int row0,
                                          int bits) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t off = ((bits >> h) & 1) != 0
                             ? static_cast<uint32_t>(row0 + L.r8 + 8 * h) * stride + L.ch * 16
                             : kOutOfBuffer;
#pragma unroll
    for (int c = 0; c < P; ++c) t.r[h][c] = __builtin_amdgcn_raw_buffer_load_b128(X.r, off + c * kRowBytes, 0, 0);
  }
}

// The mapped rows (xhat, or phi(x); zeros for rows that do not take part) into P tiles.
template <class F, int P>
__device__ __forceinline__ void stage_mapped(const Half16<P>& t, int bits, const Lane& L, float eps,
                                             unsigned char* tiles) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const bool live = ((bits >> h) & 1) != 0;
    float f[P][F::EPL];
    float ss = 0.0f;
#pragma unroll
    for (int c = 0; c < P; ++c) {
      F::unpack(t.r[h][c], f[c]);
#pragma unroll
      for (int i = 0; i < F::EPL; ++i) ss += f[c][i] * f[c][i];
    }
    const float inv = F::kMap == kMapElu1 ? 1.0f : inv_norm_or_zero(row_sum8(ss), eps, live);
#pragma unroll
    for (int c = 0; c < P; ++c) {
#pragma unroll
      for (int i = 0; i < F::EPL; ++i)
        f[c][i] = F::kMap == kMapElu1 ? (live ? elu1(f[c][i]) : 0.0f) : f[c][i] * inv;
      F::put(tiles + c * F::kTileBytes, L.r8 + 8 * h, L.ch, f[c]);
    }
  }
}

template <class F, int P>
__device__ __forceinline__ void stage_plain(const Half16<P>& t, const Lane& L, unsigned char* tiles) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < P; ++c) F::put_raw(tiles + c * F::kTileBytes, L.r8 + 8 * h, L.ch, t.r[h][c]);
}

// The blocks of the complete state that a wave ends up with: block j is piece p of x against piece
// q0 + j of y (of the transposed state when the walk was `swapped`, see below).
template <int P>
struct State {
  static constexpr int kBlocks = P * P / waves<P>();  // 1 or 2
  f32x16_t v[kBlocks];
  int p, q0;
};

// v += (x tile piece)^T (y tile piece), or with the operands exchanged, i.e. the transposed block (whose
// natural image is the one that can be written straight from the lane).
template <class F, bool SWAPPED>
__device__ __forceinline__ void add_block(f32x16_t& v, const Pieces& x, const Pieces& y) {
  v = SWAPPED ? F::mfma32(y, x, v) : F::mfma32(x, y, v);
}

// sum over the rows begin .. end-1 (those with a valid key, if `m` is given) of xhat^T y.
// The LDS area of the tiles is free afterwards (ends with a barrier).
template <class F, bool SWAPPED>
__device__ __forceinline__ void state_walk(State<2>& out, const Buffers& X, const Buffers& Y, int stride,
                                           const uint8_t* __restrict__ m, int begin, int end, float eps,
                                           const Lane& L) {
  constexpr int P = 2, kStep = 4 * TR;
  unsigned char* mine = smem + L.wave * Lds<F, P>::kPair;
  f32x16_t acc[P][P];
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int q = 0; q < P; ++q)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[p][q][i] = 0.0f;
  Half16<P> x, y;
  int row0 = begin + L.wave * TR;
  int bits = row_bits(m, row0, end, L), next_bits = row_bits(m, row0 + kStep, end, L);
  load_half(x, L, X, stride, row0, bits);
  load_half(y, L, Y, stride, row0, bits);
#pragma unroll 1
  for (; row0 < end; row0 += kStep) {
    const bool live = __builtin_amdgcn_ballot_w64(bits != 0) != 0;
    if (live) {
      stage_mapped<F, P>(x, bits, L, eps, mine);
      stage_plain<F, P>(y, L, mine + P * F::kTileBytes);
    }
    bits = next_bits;
    load_half(x, L, X, stride, row0 + kStep, bits);
    load_half(y, L, Y, stride, row0 + kStep, bits);
    next_bits = row_bits(m, row0 + 2 * kStep, end, L);
    if (live) {
      wave_lds_fence();
      const Pieces x0 = F::rows_operand(mine, L), x1 = F::rows_operand(mine + F::kTileBytes, L);
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const Pieces b = F::rows_operand(mine + (P + q) * F::kTileBytes, L);
        add_block<F, SWAPPED>(acc[0][q], x0, b);
        add_block<F, SWAPPED>(acc[1][q], x1, b);
      }
      wave_lds_fence();
    }
  }
  // wave w completes block w; the sums of the four waves are added in wave order
  out.p = L.wave >> 1;
  out.q0 = L.wave & 1;
  f32x4_t* meet = reinterpret_cast<f32x4_t*>(smem) + L.lane;  // [block][three other waves][quad][lane]
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w)
    if (w != L.wave) {
      const int slot = 3 * w + (L.wave < w ? L.wave : L.wave - 1);
#pragma unroll
      for (int g = 0; g < 4; ++g) meet[(slot * 4 + g) * 64] = quad(acc[w >> 1][w & 1], g);
    }
  __syncthreads();
  f32x16_t own = acc[0][0];
#pragma unroll
  for (int w = 1; w < 4; ++w)
    if (w == L.wave) own = acc[w >> 1][w & 1];
  f32x4_t sum[4];
#pragma unroll
  for (int w = 0; w < 4; ++w)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4_t part =
          w == L.wave ? quad(own, g) : meet[((3 * L.wave + (w < L.wave ? w : w - 1)) * 4 + g) * 64];
      sum[g] = w == 0 ? part : sum[g] + part;
    }
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int i = 0; i < 4; ++i) out.v[0][4 * g + i] = sum[g][i];
  __syncthreads();
}

template <class F, bool SWAPPED>
__device__ __forceinline__ void state_walk(State<4>& out, const Buffers& X, const Buffers& Y, int stride,
                                           const uint8_t* __restrict__ m, int begin, int end, float eps,
                                           const Lane& L) {
  constexpr int P = 4, kRound = 4 * TR;
  typedef Lds<F, P> Map;
  const int tile = L.wave & 3, part = L.wave >> 2;  // waves 0-3 stage x tiles, waves 4-7 y tiles
  unsigned char* mine = smem + tile * Map::kPair + part * P * F::kTileBytes;
  int* live_tiles = reinterpret_cast<int*>(smem + Map::kWords);
  const int p0 = L.wave & 2, q0 = 2 * (L.wave & 1);
  f32x16_t acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;
  const Buffers& mine_src = part == 0 ? X : Y;
  Half16<P> t;
  int row0 = begin + tile * TR;
  int bits = row_bits(m, row0, end, L), next_bits = row_bits(m, row0 + kRound, end, L);
  load_half(t, L, mine_src, stride, row0, bits);
#pragma unroll 1
  for (int r0 = begin; r0 < end; r0 += kRound, row0 += kRound) {
    const bool live = __builtin_amdgcn_ballot_w64(bits != 0) != 0;
    if (live) {
      if (part == 0) stage_mapped<F, P>(t, bits, L, eps, mine);
      else stage_plain<F, P>(t, L, mine);
    }
    if (part == 0 && L.lane == 0) live_tiles[tile] = live;
    bits = next_bits;
    load_half(t, L, mine_src, stride, row0 + kRound, bits);
    next_bits = row_bits(m, row0 + 2 * kRound, end, L);
    __syncthreads();
#pragma unroll 1
    for (int u = 2 * part; u < 2 * part + 2; ++u) {
      if (__builtin_amdgcn_readfirstlane(live_tiles[u]) == 0) continue;
      const unsigned char* pair = smem + u * Map::kPair;
      const Pieces x0 = F::rows_operand(pair + p0 * F::kTileBytes, L);
      const Pieces x1 = F::rows_operand(pair + (p0 + 1) * F::kTileBytes, L);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const Pieces y = F::rows_operand(pair + (P + q0 + b) * F::kTileBytes, L);
        add_block<F, SWAPPED>(acc[0][b], x0, y);
        add_block<F, SWAPPED>(acc[1][b], x1, y);
      }
    }
    __syncthreads();  // the tiles are overwritten next
  }
  // of the 2 x 2 blocks of a quadrant the first half of the workgroup completes the first row, the
  // second half the second; first half's sum + second half's sum
  out.p = p0 + part;
  out.q0 = q0;
  f32x4_t* meet = reinterpret_cast<f32x4_t*>(smem) + L.lane;  // [wave that reads][block][quad][lane]
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      meet[(((L.wave ^ 4) * 2 + b) * 4 + g) * 64] = part == 0 ? quad(acc[1][b], g) : quad(acc[0][b], g);
  __syncthreads();
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4_t own = part == 0 ? quad(acc[0][b], g) : quad(acc[1][b], g);
      const f32x4_t sum = own + meet[((L.wave * 2 + b) * 4 + g) * 64];
#pragma unroll
      for (int i = 0; i < 4; ++i) out.v[b][4 * g + i] = sum[i];
    }
  __syncthreads();
}

// The wave's blocks of scale * state into a set of images.  DIRECT: as the accumulators hold them
// (transposed images; natural ones after a swapped walk), otherwise the natural ones after a plain walk.
template <class F, int P, bool SWAPPED, bool DIRECT>
__device__ __forceinline__ void state_images(const State<P>& s, float scale, unsigned char* images, const Lane& L) {
#pragma unroll
  for (int j = 0; j < State<P>::kBlocks; ++j)
    quadrant_image<F, !DIRECT>([&](int g) { return quad(s.v[j], g); }, scale,
                               images + (P * s.p + s.q0 + j) * F::kImageBytes, L);
}

// The wave's blocks (of a plain walk) into a row-major D x D array.
template <class F, int P>
__device__ __forceinline__ void state_rows(const State<P>& s, float* __restrict__ out, const Lane& L) {
  constexpr int D = P * F::D;
#pragma unroll
  for (int j = 0; j < State<P>::kBlocks; ++j)
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        out[(s.p * F::D + F::run_row(g, L) + i) * D + (s.q0 + j) * F::D + F::run_col(L)] = s.v[j][4 * g + i];
}

// ---- apply ----------------------------------------------------------------------------------------------

template <int P>
__device__ __forceinline__ void floats_of(const OwnRaw<P>& t, int c, float (&f)[8]) {
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) f[4 * j + i] = __uint_as_float(t.r[c][j][i]);
}

// 1/r of the lane's row under the cosine map (0 for a row that does not take part), 1 under ELU + 1.
template <class F, int P>
__device__ __forceinline__ float own_factor(const OwnRaw<P>& t, float eps, bool live, const Lane& L) {
  if (F::kMap == kMapElu1) return 1.0f;
  float ss = 0.0f;
#pragma unroll
  for (int c = 0; c < P; ++c) {
    float f[8];
    floats_of(t, c, f);
#pragma unroll
    for (int i = 0; i < 8; ++i) ss += f[i] * f[i];
  }
  return inv_norm_or_zero(row_sum_groups(ss, L), eps, live);
}

// The rows as they enter a product whose result is multiplied by own_factor(): raw, or phi(x).
template <class F, int P>
__device__ __forceinline__ void own_mapped(const OwnRaw<P>& t, bool live, typename F::TileRows (&x)[P]) {
#pragma unroll
  for (int c = 0; c < P; ++c) {
    float f[8];
    floats_of(t, c, f);
    if (F::kMap == kMapElu1) {
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = live ? elu1(f[i]) : 0.0f;
    }
    x[c].set(f);
  }
}

// out = sum_c X[c] W(first + c * step)
template <class F, int P>
__device__ __forceinline__ void product(const typename F::TileRows (&X)[P], const unsigned char* images, int first,
                                        int step, const Lane& L, float (&out)[8]) {
  f32x4_t a[F::NT];
#pragma unroll
  for (int nt = 0; nt < F::NT; ++nt) a[nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < P; ++c) {
    typename F::Operand W;
    W.load(images + (first + c * step) * F::kImageBytes, L);
    F::apply_onto(X[c], W, a);
  }
  product_rows<F>(a, out);
}

template <class F, int P>
__device__ __forceinline__ void store_piece(unsigned char* out, int c, int row, int end, int stride, const Lane& L,
                                            const float (&o)[8]) {
  if (row < end)
    store_product_row<F, kStoreStreamed>(out + c * kRowBytes, row, RowAddr{stride, kRowBytes}, L, o);
}

template <class F, int P>
__device__ __forceinline__ void store_zeros(unsigned char* out, int row, int end, int stride, const Lane& L) {
  float z[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = 0.0f;
#pragma unroll
  for (int c = 0; c < P; ++c) store_piece<F, P>(out, c, row, end, stride, L, z);
}

// One tile of out = (x rows) M (contraction over the rows of M; `images`: the transposed ones).
template <class F, int P>
__device__ __forceinline__ void plain_tile(const OwnRaw<P>& raw, bool live, float inv, const unsigned char* images,
                                           unsigned char* out, int row, int end, int stride, const Lane& L) {
  typename F::TileRows x[P];
  own_mapped<F, P>(raw, live, x);
#pragma unroll
  for (int q = 0; q < P; ++q) {
    float o[8];
    product<F, P>(x, images, q, P, L, o);
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] *= inv;
    store_piece<F, P>(out, q, row, end, stride, L, o);
  }
}

// One tile of out = J (y rows) M^T, J the derivative of the map at the x rows (contraction over the
// columns of M; `images`: the natural ones).  Returns mapped x . (y M^T) of the lane's row.
template <class F, int P>
__device__ __forceinline__ float projected_tile(const OwnRaw<P>& x, const OwnRaw<P>& y, bool live, float inv,
                                                const unsigned char* images, unsigned char* out, int row, int end,
                                                int stride, const Lane& L, bool want_dot) {
  float g[P][8];
  {
    typename F::TileRows Y[P];
    own_rows<F, P>(y, Y);
#pragma unroll
    for (int p = 0; p < P; ++p) product<F, P>(Y, images, P * p, 1, L, g[p]);
  }
  float dot = 0.0f;
  if (F::kMap != kMapElu1 || want_dot) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      float f[8];
      floats_of(x, p, f);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        dot += (F::kMap == kMapElu1 ? (live ? elu1(f[i]) : 0.0f) : f[i] * inv) * g[p][i];
    }
    dot = row_sum_groups(dot, L);
  }
#pragma unroll
  for (int p = 0; p < P; ++p) {
    float f[8];
    floats_of(x, p, f);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      g[p][i] = F::kMap == kMapElu1 ? g[p][i] * fminf(elu1(f[i]), 1.0f) : (g[p][i] - f[i] * inv * dot) * inv;
    store_piece<F, P>(out, p, row, end, stride, L, g[p]);
  }
  return dot;
}

struct Rows16 {  // the tiles of a wave: first, first + step, ... below end
  int begin, end, stride;
};

template <class F, int P>
__device__ __forceinline__ bool own_live(const uint8_t* keys, int row, int end) {
  return row < end && (keys == nullptr || keys[row] != 0);
}

// O, or dV alone.  `first`: the wave's first tile, already requested.
template <class F, int P>
__device__ __forceinline__ void apply_plain(const Buffers& X, const uint8_t* keys, const Rows16 r, float eps,
                                            const unsigned char* images, unsigned char* out, const Lane& L,
                                            const OwnRaw<P>& first) {
  constexpr int kStep = waves<P>() * TR;
  const RowAddr addr{r.stride, P * kRowBytes};
  OwnRaw<P> next = first;
  bool next_live = own_live<F, P>(keys, r.begin + L.wave * TR + L.i16, r.end);
#pragma unroll 1
  for (int row0 = r.begin + L.wave * TR; row0 < r.end; row0 += kStep) {
    const OwnRaw<P> cur = next;
    const bool live = next_live;
    next_live = own_live<F, P>(keys, row0 + kStep + L.i16, r.end);
    load_own<P>(next, L, X, addr, row0 + kStep, next_live);
    const int row = row0 + L.i16;
    if (__builtin_amdgcn_ballot_w64(live) == 0) {
      store_zeros<F, P>(out, row, r.end, r.stride, L);
      continue;
    }
    plain_tile<F, P>(cur, live, own_factor<F, P>(cur, eps, live, L), images, out, row, r.end, r.stride, L);
  }
}

// dQ, or dK alone.  Returns this lane's share of sum_i x_i . (y_i M^T).
template <class F, int P>
__device__ __forceinline__ float apply_projected(const Buffers& X, const Buffers& Y, const uint8_t* keys,
                                                 const Rows16 r, float eps, const unsigned char* images,
                                                 unsigned char* out, const Lane& L, const OwnRaw<P>& first_x,
                                                 const OwnRaw<P>& first_y, bool want_dot) {
  constexpr int kStep = waves<P>() * TR;
  const RowAddr addr{r.stride, P * kRowBytes};
  float dots = 0.0f;
  OwnRaw<P> nx = first_x, ny = first_y;
  bool next_live = own_live<F, P>(keys, r.begin + L.wave * TR + L.i16, r.end);
#pragma unroll 1
  for (int row0 = r.begin + L.wave * TR; row0 < r.end; row0 += kStep) {
    const OwnRaw<P> x = nx, y = ny;
    const bool live = next_live;
    next_live = own_live<F, P>(keys, row0 + kStep + L.i16, r.end);
    load_own<P>(nx, L, X, addr, row0 + kStep, next_live);
    load_own<P>(ny, L, Y, addr, row0 + kStep, next_live);
    const int row = row0 + L.i16;
    if (__builtin_amdgcn_ballot_w64(live) == 0) {
      store_zeros<F, P>(out, row, r.end, r.stride, L);
      continue;
    }
    const float inv = own_factor<F, P>(x, eps, live, L);
    const float dot = projected_tile<F, P>(x, y, live, inv, images, out, row, r.end, r.stride, L, want_dot);
    if (L.g16 == 0) dots += dot;
  }
  return dots;
}

// dV and dK together, both image sets being there: K and V are read once.
template <class F, int P>
__device__ __forceinline__ void apply_both(const Buffers& K, const Buffers& V, const uint8_t* keys, const Rows16 r,
                                           float eps, const unsigned char* transposed, const unsigned char* natural,
                                           unsigned char* dV, unsigned char* dK, const Lane& L,
                                           const OwnRaw<P>& first_k, const OwnRaw<P>& first_v) {
  constexpr int kStep = waves<P>() * TR;
  const RowAddr addr{r.stride, P * kRowBytes};
  OwnRaw<P> nk = first_k, nv = first_v;
  bool next_live = own_live<F, P>(keys, r.begin + L.wave * TR + L.i16, r.end);
#pragma unroll 1
  for (int row0 = r.begin + L.wave * TR; row0 < r.end; row0 += kStep) {
    const OwnRaw<P> k = nk, v = nv;
    const bool live = next_live;
    next_live = own_live<F, P>(keys, row0 + kStep + L.i16, r.end);
    load_own<P>(nk, L, K, addr, row0 + kStep, next_live);
    load_own<P>(nv, L, V, addr, row0 + kStep, next_live);
    const int row = row0 + L.i16;
    if (__builtin_amdgcn_ballot_w64(live) == 0) {
      store_zeros<F, P>(dV, row, r.end, r.stride, L);
      store_zeros<F, P>(dK, row, r.end, r.stride, L);
      continue;
    }
    const float inv = own_factor<F, P>(k, eps, live, L);
    plain_tile<F, P>(k, live, inv, transposed, dV, row, r.end, r.stride, L);
    projected_tile<F, P>(k, v, live, inv, natural, dK, row, r.end, r.stride, L, false);
  }
}

// ---- one launch per direction ------------------------------------------------------------------------------

template <class F, int P>
__global__ __launch_bounds__(64 * waves<P>(), P == 2 ? 3 : 2) void fused_fwd_kernel(const Args a) {
  typedef Lds<F, P> Map;
  constexpr int D = P * F::D;
  const Lane L;
  const int bh = blockIdx.x, N = a.N, stride = a.st.row.stride;
  const size_t base = a.st.slice_base(bh, a.H);
  State<P> s;
  {
    const Buffers K(a.K + base, N, a.st.row), V(a.V + base, N, a.st.row);
    state_walk<F, false>(s, K, V, stride, a.keys_of(bh), 0, N, a.eps, L);
  }
  // the first tile of Q travels while the images are made
  const Buffers Q(a.Q + base, N, a.st.row);
  OwnRaw<P> first;
  load_own<P>(first, L, Q, a.st.row, L.wave * TR, L.wave * TR + L.i16 < N);
  state_images<F, P, false, true>(s, a.scale_of(bh), smem, L);
  if (a.kept != nullptr) state_rows<F, P>(s, a.kept + static_cast<size_t>(bh) * D * D, L);
  __syncthreads();
  apply_plain<F, P>(Q, nullptr, Rows16{0, N, stride}, a.eps, smem, a.O + base, L, first);
}

template <class F, int P>
__global__ __launch_bounds__(64 * waves<P>(), P == 2 ? 3 : 2) void fused_bwd_kernel(const Args a) {
  typedef Lds<F, P> Map;
  const Lane L;
  // workgroups go to the XCDs round-robin: the two roles of a slice are eight apart, on one XCD
  const int bh = (blockIdx.x >> 4) * 8 + (blockIdx.x & 7);
  const bool second = ((blockIdx.x >> 3) & 1) != 0;
  if (bh >= a.slices) return;
  const int N = a.N, stride = a.st.row.stride;
  const size_t base = a.st.slice_base(bh, a.H);
  const uint8_t* keys = a.keys_of(bh);
  const float scale = a.scale_of(bh);
  const Buffers Q(a.Q + base, N, a.st.row), K(a.K + base, N, a.st.row);
  const Buffers V(a.V + base, N, a.st.row), dO(a.dO + base, N, a.st.row);
  const int row = L.wave * TR + L.i16;
  const Rows16 all{0, N, stride};
  State<P> s;
  OwnRaw<P> fx, fy;
  if (!second) {
    state_walk<F, true>(s, K, V, stride, keys, 0, N, a.eps, L);
    load_own<P>(fx, L, Q, a.st.row, L.wave * TR, row < N);
    load_own<P>(fy, L, dO, a.st.row, L.wave * TR, row < N);
    state_images<F, P, true, true>(s, scale, smem, L);
    __syncthreads();
    float dots = apply_projected<F, P>(Q, dO, nullptr, all, a.eps, smem, a.dQ + base, L, fx, fy, a.dlog != nullptr);
    if (a.dlog != nullptr) {  // sum_i dO_i . O_i = sum_i qhat_i . (scale dO_i S^T), in a fixed order
      float* partial = reinterpret_cast<float*>(smem + Map::kWords);
      dots = wave_sum(dots);
      if (L.lane == 0) partial[L.wave] = dots;
      __syncthreads();
      if (threadIdx.x == 0) {
        float sum = 0.0f;
        for (int w = 0; w < waves<P>(); ++w) sum += partial[w];
        a.dlog[bh] = sum;
      }
    }
    return;
  }
  state_walk<F, false>(s, Q, dO, stride, nullptr, 0, N, a.eps, L);
  const bool live = own_live<F, P>(keys, row, N);
  load_own<P>(fx, L, K, a.st.row, L.wave * TR, live);
  if (P == 2) {
    load_own<P>(fy, L, V, a.st.row, L.wave * TR, live);
    state_images<F, P, false, true>(s, scale, smem, L);
    state_images<F, P, false, false>(s, scale, smem + Map::kSet, L);
    __syncthreads();
    apply_both<F, P>(K, V, keys, all, a.eps, smem, smem + Map::kSet, a.dV + base, a.dK + base, L, fx, fy);
  } else {
    state_images<F, P, false, true>(s, scale, smem, L);
    __syncthreads();
    apply_plain<F, P>(K, keys, all, a.eps, smem, a.dV + base, L, fx);
    load_own<P>(fx, L, K, a.st.row, L.wave * TR, live);
    load_own<P>(fy, L, V, a.st.row, L.wave * TR, live);
    __syncthreads();  // nobody reads the transposed images any more
    state_images<F, P, false, false>(s, scale, smem, L);
    __syncthreads();
    apply_projected<F, P>(K, V, keys, all, a.eps, smem, a.dK + base, L, fx, fy, false);
  }
}

// ---- three launches --------------------------------------------------------------------------------------------

// grid (slices * splits, 1 or 2); blockIdx.y == 1 reduces (Q, dO) instead of (K, V) under the key mask.
// Partial states: row-major D x D floats per workgroup, the second kind behind all of the first.
template <class F, int P>
__global__ __launch_bounds__(64 * waves<P>(), P == 2 ? 3 : 2) void state_kernel(const Args a, float* __restrict__ ws) {
  constexpr int D = P * F::D;
  const Lane L;
  const int split = blockIdx.x % a.splits, bh = blockIdx.x / a.splits;
  const bool second = blockIdx.y == 1;
  const size_t base = a.st.slice_base(bh, a.H);
  const Buffers X((second ? a.Q : a.K) + base, a.N, a.st.row), Y((second ? a.dO : a.V) + base, a.N, a.st.row);
  const int begin = split * a.rows_per_split;
  const int end = a.N < begin + a.rows_per_split ? a.N : begin + a.rows_per_split;
  State<P> s;
  state_walk<F, false>(s, X, Y, a.st.row.stride, second ? nullptr : a.keys_of(bh), begin, end, a.eps, L);
  state_rows<F, P>(s, ws + (static_cast<size_t>(blockIdx.y) * gridDim.x + blockIdx.x) * D * D, L);
}

// The images of scale * M (M: a complete state in global memory, row-major D x D): block (p, q) at
// P p + q, natural op[m][n] or transposed op[n][m] = M[p 32 + m][q 32 + n].
template <class F, int P, bool TRANSPOSED>
__device__ __forceinline__ void build_images(const float* __restrict__ M, float scale, unsigned char* images) {
  constexpr int D = P * F::D, kThreads = 64 * waves<P>(), kPairs = D * D / 2, kBatch = 8;
  static_assert(kPairs % (kBatch * kThreads) == 0, "state size");
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
        const float2 v = *reinterpret_cast<const float2*>(M + e / (D / 2) * D + 2 * (e % (D / 2)));
        v0[j] = v.x;
        v1[j] = v.y;
      }
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int e = e0 + j * kThreads;
      const int m = TRANSPOSED ? 2 * (e / D) : e / (D / 2);
      const int n = TRANSPOSED ? e % D : 2 * (e % (D / 2));
      unsigned char* image = images + (P * (m / F::D) + n / F::D) * F::kImageBytes;
      if (TRANSPOSED) F::write_image_pair(image, n % F::D, m % F::D, v0[j] * scale, v1[j] * scale);
      else F::write_image_pair(image, m % F::D, n % F::D, v0[j] * scale, v1[j] * scale);
    }
  }
}

template <class F, int P>
__global__ __launch_bounds__(64 * waves<P>(), P == 2 ? 3 : 2) void apply_fwd_kernel(const Args a) {
  constexpr int D = P * F::D;
  const Lane L;
  const int split = blockIdx.x % a.splits, bh = blockIdx.x / a.splits;
  const size_t base = a.st.slice_base(bh, a.H);
  const int begin = split * a.rows_per_split;
  const int end = a.N < begin + a.rows_per_split ? a.N : begin + a.rows_per_split;
  const int row0 = begin + L.wave * TR;
  const Buffers Q(a.Q + base, a.N, a.st.row);
  OwnRaw<P> first;
  load_own<P>(first, L, Q, a.st.row, row0, row0 + L.i16 < end);
  build_images<F, P, true>(a.states + static_cast<size_t>(bh) * D * D, a.scale_of(bh), smem);
  __syncthreads();
  apply_plain<F, P>(Q, nullptr, Rows16{begin, end, a.st.row.stride}, a.eps, smem, a.O + base, L, first);
}

// blockIdx.y: 0 dQ, 1 dV, 2 dK
template <class F, int P>
__global__ __launch_bounds__(64 * waves<P>(), P == 2 ? 3 : 2) void apply_bwd_kernel(const Args a) {
  constexpr int D = P * F::D;
  const Lane L;
  const int split = blockIdx.x % a.splits, bh = blockIdx.x / a.splits, role = blockIdx.y;
  const size_t base = a.st.slice_base(bh, a.H);
  const int begin = split * a.rows_per_split;
  const int end = a.N < begin + a.rows_per_split ? a.N : begin + a.rows_per_split;
  const int row0 = begin + L.wave * TR;
  const Rows16 rows{begin, end, a.st.row.stride};
  const uint8_t* keys = role == 0 ? nullptr : a.keys_of(bh);
  const Buffers X((role == 0 ? a.Q : a.K) + base, a.N, a.st.row), Y((role == 0 ? a.dO : a.V) + base, a.N, a.st.row);
  const float* M = (role == 0 ? a.states : a.dstates) + static_cast<size_t>(bh) * D * D;
  const bool live = own_live<F, P>(keys, row0 + L.i16, end);
  OwnRaw<P> fx, fy;
  load_own<P>(fx, L, X, a.st.row, row0, live);
  if (role == 1) {
    build_images<F, P, true>(M, a.scale_of(bh), smem);
    __syncthreads();
    apply_plain<F, P>(X, keys, rows, a.eps, smem, a.dV + base, L, fx);
  } else {
    load_own<P>(fy, L, Y, a.st.row, row0, live);
    build_images<F, P, false>(M, a.scale_of(bh), smem);
    __syncthreads();
    apply_projected<F, P>(X, Y, keys, rows, a.eps, smem, (role == 0 ? a.dQ : a.dK) + base, L, fx, fy, false);
  }
}

// ---- host side ---------------------------------------------------------------------------------------------------

Args make_args(const Problem& p, const Plan& plan) {
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
  a.scale = p.scale;
  a.eps = p.eps;
  a.slice_scale = p.slice_scale;
  a.kept = p.saved_state;
  a.dlog = p.dlog_scale;
  a.splits = plan.splits;
  a.rows_per_split = plan.rows_per_split;
  a.st = Strides{p.stride_batch * 4, p.stride_head * 4,
                 RowAddr{static_cast<int>(p.stride_row * 4), static_cast<int>(p.D * 4)}};
  return a;
}

template <class Kernel, class... Extra>
hipError_t launch(Kernel kernel, dim3 grid, int threads, int lds, const Problem& p, const Args& a, Extra... extra) {
  const hipError_t err = grant_dynamic_lds(reinterpret_cast<const void*>(kernel), lds);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, p.stream, a, extra...);
  return hipGetLastError();
}

enum Kind { kFused, kStates, kApply };

template <class F, int P>
hipError_t run(Kind kind, const Problem& p, const Args& a, bool bwd) {
  constexpr int threads = 64 * waves<P>(), lds = Lds<F, P>::kBytes;
  static_assert(lds <= (P == 2 ? 160 * 1024 / 3 : 160 * 1024), "three workgroups per compute unit, or one");
  const unsigned slices = static_cast<unsigned>(a.slices);
  if (kind == kFused)
    return bwd ? launch(fused_bwd_kernel<F, P>, dim3((slices + 7) / 8 * 16), threads, lds, p, a)
               : launch(fused_fwd_kernel<F, P>, dim3(slices), threads, lds, p, a);
  const unsigned blocks = slices * a.splits;
  if (kind == kStates) return launch(state_kernel<F, P>, dim3(blocks, bwd ? 2 : 1), threads, lds, p, a, p.workspace);
  return bwd ? launch(apply_bwd_kernel<F, P>, dim3(blocks, 3), threads, lds, p, a)
             : launch(apply_fwd_kernel<F, P>, dim3(blocks), threads, lds, p, a);
}

hipError_t dispatch(Kind kind, const Problem& p, const Args& a, bool bwd) {
  typedef WithElu1<F32x32> Elu;
  if (p.feature_map == kMapElu1)
    return p.D == 64 ? run<Elu, 2>(kind, p, a, bwd) : run<Elu, 4>(kind, p, a, bwd);
  return p.D == 64 ? run<F32x32, 2>(kind, p, a, bwd) : run<F32x32, 4>(kind, p, a, bwd);
}

}  // namespace wide32
}  // namespace

hipError_t launch_wide32_states(const Problem& p, const Plan& plan, bool bwd) {
  return wide32::dispatch(wide32::kStates, p, wide32::make_args(p, plan), bwd);
}

hipError_t launch_wide32_fused(const Problem& p, const Plan& plan, bool bwd) {
  return wide32::dispatch(wide32::kFused, p, wide32::make_args(p, plan), bwd);
}

hipError_t launch_wide32_apply(const Problem& p, const Plan& plan, const float* states, const float* dstates,
                               bool bwd) {
  wide32::Args a = wide32::make_args(p, plan);
  a.states = states;
  a.dstates = dstates;
  return wide32::dispatch(wide32::kApply, p, a, bwd);
}

}  // namespace cotten
