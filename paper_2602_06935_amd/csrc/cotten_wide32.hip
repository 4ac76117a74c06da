// fp32 rows of 256 and 512 bytes (d_h = 64 and 128) on the matrix cores: a row in P = 2 or 4 pieces of
// 128 bytes, a state in P x P blocks of 32 x 32, every product as six products of bf16 pieces
// (F32x32 in cotten_mfma_core.h).
//
//     S[p][q]  = sum_j khat_j[piece p]^T v_j[piece q]                     (state walk)
//     O[q]     = sum_p Qhat[piece p] S[p][q]       likewise dQ, dK, dV    (apply)
//
// State walk: the rows go through LDS, where the matrix cores read them transposed, cut into
// pieces once on the way.
//   P = 2, four waves   a wave adds its own tiles to a state of its own (no barriers), the four sums
//                       meet at the end
//   P = 2, eight waves  (few workgroups) rounds of 128 rows, a wave adds the tiles of its half of the
//                       workgroup to one block, the two sums of a block meet at the end
//   P = 4, eight waves  rounds of 32 rows in two buffers, a wave adds one of the two tiles of a round to a
//                       quadrant of 2 x 2 blocks, the two sums of a quadrant meet at the end
// Apply: a wave loads its own rows straight in the layout of the products (no LDS), the state is
// read from operand images that lie over the tiles of the walk.
//
// A sequence that is not cut takes one launch per direction (d_h = 128: up to 256 slices, in the backward 128; most of what
// has more goes to cotten_columns.hip) and the state never leaves the compute unit; the backward has two roles, side by side on one XCD, each of which reads all four tensors:
//   S from (K, V), then dQ;      dS from (Q, dO), then dV and dK
// A cut one takes three launches: partial states into the caller's workspace, their sum in split
// order (reduce_states_kernel), apply (backward: three roles).
#include <type_traits>

#include "cotten_launch.h"
#include "cotten_mfma_core.h"

namespace cotten {
namespace {
namespace wide32 {

using namespace mfma;

extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

// LDS: the tiles of the state walk; over them, once the state is complete, the sums that meet and
// then the operand images; behind them a few words.
template <class F, int P, int WAVES>
struct Lds {
  static constexpr int kPair = 2 * P * F::kTileBytes;   // [x pieces | y pieces] of 16 rows
  static constexpr int kPairs = P == 2 ? WAVES : 4;     // one per wave; P = 4: two rounds of 32 rows
  static constexpr int kTiles = kPairs * kPair;
  static constexpr int kSet = P * P * F::kImageBytes;
  static constexpr int kSets = P == 2 ? 2 : 1;          // image sets there is room for
  static constexpr int kWords = kTiles;
  static_assert(kSets * kSet <= kTiles, "the images lie over the tiles");
  static constexpr int kBytes = kWords + 64;
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
  float top = 0.0f;  // (phi(x) is infinite where x is)
  if (F::kMap == kMapElu1) {
#pragma unroll
    for (int c = 0; c < P; ++c) top = F::largest_raw(t.r[0][c], F::largest_raw(t.r[1][c], top));
  }
  write_pieces<F>(top, [&](auto inf) {
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
          f[c][i] = F::kMap == kMapElu1 ? elu1_or_zero(f[c][i], live) : f[c][i] * inv;
        F::template put<decltype(inf)::value>(tiles + c * F::kTileBytes, L.r8 + 8 * h, L.ch, f[c]);
      }
    }
  });
}

template <class F, int P>
__device__ __forceinline__ void stage_plain(const Half16<P>& t, const Lane& L, unsigned char* tiles) {
  float top = 0.0f;
#pragma unroll
  for (int c = 0; c < P; ++c) top = F::largest_raw(t.r[0][c], F::largest_raw(t.r[1][c], top));
  write_pieces<F>(top, [&](auto inf) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < P; ++c)
        F::template put_raw<decltype(inf)::value>(tiles + c * F::kTileBytes, L.r8 + 8 * h, L.ch, t.r[h][c]);
  });
}

// The blocks of the complete state that a wave ends up with: block j is piece p of the left rows
// against piece q0 + j of the right ones.  With two groups of four waves the second has none.
template <class F, int P>
struct State {
  static constexpr int kBlocks = P == 2 ? 1 : 2;
  typename F::Acc v[kBlocks];
  int p, q0;
  bool here;
};

// The first row at which a key is valid, down to a multiple of 16 (N if there is none; 0 without looking
// for long sequences): a left-padded history of at most 512 rows is walked from there (rows of two
// pieces: the live tiles are dealt evenly to the waves; 512 slices x 200 rows, forward 25.5 -> 24.7 us).
__device__ __forceinline__ int first_live_tile(const uint8_t* __restrict__ m, int N, const Lane& L) {
  constexpr int kMost = 512;
  if (m == nullptr || N > kMost) return 0;
  int lo = N;
#pragma unroll
  for (int i = kMost / 64 - 1; i >= 0; --i) {
    const int row = 64 * i + L.lane;
    const uint64_t set = __builtin_amdgcn_ballot_w64(row < N && m[row < N ? row : 0] != 0);
    if (set != 0) lo = 64 * i + __builtin_ctzll(set);
  }
  return lo == N ? N : lo & ~(TR - 1);
}

template <int P>
__device__ __forceinline__ int walk_begin(const uint8_t* __restrict__ m, int N, const Lane& L) {
  // (up to 64 rows every wave has its one tile requested at once, and looking first is a trip to memory)
  return P == 4 || N <= 4 * TR ? 0 : first_live_tile(m, N, L);
}

// The walks: sum over the rows begin .. end-1 (those with a valid key, if `m` is given) of xhat^T y - or,
// SWAPPED, y^T xhat, the transposed state, whose natural images are the ones that can be written
// straight from the lanes.  The LDS area of the tiles is free afterwards (they end with a barrier).
// `request` asks for what comes next, once the rows have arrived and only the sums are left to meet.

// P = 2, eight waves: one block per wave (wave & 3) and group of four waves; every wave stages one tile
// pair per round, a group adds its own four.
template <class F, bool SWAPPED, class Request>
__device__ __forceinline__ void walk_shared(State<F, 2>& out, const Buffers& X, const Buffers& Y, int stride,
                                            const uint8_t* __restrict__ m, int begin, int end, float eps,
                                            const Lane& L, Request&& request) {
  constexpr int P = 2, WAVES = 8, kRound = WAVES * TR;
  typedef Lds<F, P, WAVES> Map;
  const int group = L.wave >> 2, p = (L.wave >> 1) & 1, q = L.wave & 1;
  unsigned char* mine = smem + L.wave * Map::kPair;
  int* live_tiles = reinterpret_cast<int*>(smem + Map::kWords);
  const int left = (SWAPPED ? P + p : p) * F::kTileBytes, right = (SWAPPED ? q : P + q) * F::kTileBytes;
  // a sum over more than eight tiles is a sum of sums over eight (two rounds of the wave's four): error of dK against
  // float64, 100 slices x 1500 rows, 2.0e-7 as one sum
  typename F::Acc& acc = out.v[0];
  typename F::Acc sums;
  acc.zero();
  sums.zero();
  out.p = p;
  out.q0 = q;
  out.here = group == 0;
  Half16<P> x, y;
  int row0 = begin + L.wave * TR;
  int bits = row_bits(m, row0, end, L), next_bits = row_bits(m, row0 + kRound, end, L);
  load_half(x, L, X, stride, row0, bits);
  load_half(y, L, Y, stride, row0, bits);
  bool odd = false;
#pragma unroll 1
  for (int r0 = begin; r0 < end; r0 += kRound, row0 += kRound) {
    const bool live = __builtin_amdgcn_ballot_w64(bits != 0) != 0;
    if (live) {
      stage_mapped<F, P>(x, bits, L, eps, mine);
      stage_plain<F, P>(y, L, mine + P * F::kTileBytes);
    }
    if (L.lane == 0) live_tiles[L.wave] = live;
    bits = next_bits;
    load_half(x, L, X, stride, row0 + kRound, bits);
    load_half(y, L, Y, stride, row0 + kRound, bits);
    next_bits = row_bits(m, row0 + 2 * kRound, end, L);
    __syncthreads();
    int flags = 0;
#pragma unroll
    for (int t = 0; t < 4; ++t) flags |= (live_tiles[4 * group + t] != 0) << t;
    flags = __builtin_amdgcn_readfirstlane(flags);
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if ((flags >> t) & 1) {
        const unsigned char* pair = smem + (4 * group + t) * Map::kPair;
        acc.mfma(pair + left, pair + right, L);
      }
    if (F::kApart && odd) {
#pragma unroll
      for (int g = 0; g < F::Acc::kGroups; ++g) sums.add_group(g, acc.group(g));
      acc.zero();
    }
    odd = !odd;
    __syncthreads();  // the tiles are overwritten next
  }
  if (F::kApart) {
#pragma unroll
    for (int g = 0; g < F::Acc::kGroups; ++g) sums.add_group(g, acc.group(g));
    acc = sums;
  }
  request();
  {  // first group's sum + second group's sum
    static_assert(4 * F::Acc::kGroups * 64 * 16 <= Map::kTiles, "the sums meet in the tiles");
    f32x4_t* meet = reinterpret_cast<f32x4_t*>(smem) + (L.wave & 3) * F::Acc::kGroups * 64 + L.lane;
    if (group == 1) {
#pragma unroll
      for (int g = 0; g < F::Acc::kGroups; ++g) meet[g * 64] = acc.group(g);
    }
    __syncthreads();
    if (group == 0) {
#pragma unroll
      for (int g = 0; g < F::Acc::kGroups; ++g) acc.add_group(g, meet[g * 64]);
    }
    __syncthreads();
  }
}

// P = 2, four waves: a wave adds its own tiles (every fourth) to a state of its own.
template <class F, bool SWAPPED, class Request>
__device__ __forceinline__ void walk_private(State<F, 2>& out, const Buffers& X, const Buffers& Y, int stride,
                                             const uint8_t* __restrict__ m, int begin, int end, float eps,
                                             const Lane& L, Request&& request) {
  constexpr int P = 2, kStep = 4 * TR;
  typedef Lds<F, P, 4> Map;
  unsigned char* mine = smem + L.wave * Map::kPair;
  const unsigned char* left = mine + (SWAPPED ? P : 0) * F::kTileBytes;
  const unsigned char* right = mine + (SWAPPED ? 0 : P) * F::kTileBytes;
  typename F::Acc acc[P][P];
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int q = 0; q < P; ++q) acc[p][q].zero();
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
      const Pieces l0 = F::rows_operand(left, L), l1 = F::rows_operand(left + F::kTileBytes, L);
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const Pieces r = F::rows_operand(right + q * F::kTileBytes, L);
        acc[0][q].add_lean(l0, r);
        acc[1][q].add_lean(l1, r);
      }
      wave_lds_fence();
    }
  }
  request();
  // wave w completes block w; the sums of the four waves are added in wave order
  out.p = L.wave >> 1;
  out.q0 = L.wave & 1;
  out.here = true;
  f32x4_t* meet = reinterpret_cast<f32x4_t*>(smem) + L.lane;  // [block][three other waves][quad][lane]
  static_assert(12 * 4 * 64 * 16 <= Map::kTiles, "the sums meet in the tiles");
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w)
    if (w != L.wave) {
      const int slot = 3 * w + (L.wave < w ? L.wave : L.wave - 1);
#pragma unroll
      for (int g = 0; g < 4; ++g) meet[(slot * 4 + g) * 64] = acc[w >> 1][w & 1].group(g);
    }
  __syncthreads();
  typename F::Acc own = acc[0][0];
#pragma unroll
  for (int w = 1; w < 4; ++w)
    if (w == L.wave) own = acc[w >> 1][w & 1];
  f32x4_t sum[4];
#pragma unroll
  for (int w = 0; w < 4; ++w)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4_t part =
          w == L.wave ? own.group(g) : meet[((3 * L.wave + (w < L.wave ? w : w - 1)) * 4 + g) * 64];
      sum[g] = w == 0 ? part : sum[g] + part;
    }
  out.v[0].zero();
#pragma unroll
  for (int g = 0; g < 4; ++g) out.v[0].add_group(g, sum[g]);
  __syncthreads();
}

// P = 4: rounds of 32 rows in two LDS buffers.  Waves 0-3 stage 8 rows of x each, waves 4-7 8 rows of y;
// a wave adds one of the two tiles of a round to its quadrant of 2 x 2 blocks.  One barrier per round; of
// the two waves of a SIMD one stages the next round (vector units) before, the other after its products
// (matrix cores), so that both are busy.  (All waves staging, then all multiplying: 28 k of the 56 k cycles of
// a slice of 200 rows; forward of 256 slices x 1000 rows 124 -> 117 us, of 16 slices x 200 24.4 -> 22.5.)
template <class F, bool SWAPPED, class Request>
__device__ __forceinline__ void walk_quadrants(State<F, 4>& out, const Buffers& X, const Buffers& Y, int stride,
                                               const uint8_t* __restrict__ m, int begin, int end, float eps,
                                               const Lane& L, Request&& request) {
  constexpr int P = 4, kRound = 2 * TR;
  typedef Lds<F, P, 8> Map;
  constexpr int kBuffer = 2 * Map::kPair;
  const int part = L.wave >> 2;  // what the wave stages (x or y), and the tile of a round that it adds
  const int row = 16 * ((L.wave >> 1) & 1) + 8 * (L.wave & 1) + L.r8;  // of a round, that it stages
  unsigned char* mine = smem + (row >> 4) * Map::kPair + part * P * F::kTileBytes;
  int* live_halves = reinterpret_cast<int*>(smem + Map::kWords);  // [buffer][wave 0-3]
  const int p0 = L.wave & 2, q0 = 2 * (L.wave & 1);
  const int left = part * Map::kPair + ((SWAPPED ? P : 0) + p0) * F::kTileBytes;
  const int right = part * Map::kPair + ((SWAPPED ? 0 : P) + q0) * F::kTileBytes;
  typename F::Acc acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b].zero();
  const Buffers& source = part == 0 ? X : Y;
  u32x4_t raw[2][P];  // rounds on their way (two ahead of the one being staged)
  bool live[2];
  const auto row_at = [&](int r0) { return r0 + row < end && (m == nullptr || m[r0 + row] != 0); };
  const auto load = [&](u32x4_t (&t)[P], int r0, bool on) {
    const uint32_t off = on ? static_cast<uint32_t>(r0 + row) * stride + L.ch * 16 : kOutOfBuffer;
#pragma unroll
    for (int c = 0; c < P; ++c) t[c] = __builtin_amdgcn_raw_buffer_load_b128(source.r, off + c * kRowBytes, 0, 0);
  };
  const auto stage = [&](const u32x4_t (&t)[P], bool on, int buffer) {
    float f[P][F::EPL];
    float ss = 0.0f;
#pragma unroll
    for (int c = 0; c < P; ++c) F::unpack(t[c], f[c]);
    if (part == 0) {
#pragma unroll
      for (int c = 0; c < P; ++c)
#pragma unroll
        for (int i = 0; i < F::EPL; ++i) ss += f[c][i] * f[c][i];
      const float inv = F::kMap == kMapElu1 ? 1.0f : inv_norm_or_zero(row_sum8(ss), eps, on);
#pragma unroll
      for (int c = 0; c < P; ++c)
#pragma unroll
        for (int i = 0; i < F::EPL; ++i)
          f[c][i] = F::kMap == kMapElu1 ? elu1_or_zero(f[c][i], on) : f[c][i] * inv;
      const bool any = __builtin_amdgcn_ballot_w64(on) != 0;
      if (L.lane == 0) live_halves[4 * buffer + L.wave] = any;
    }
    float top = 0.0f;
    if (F::kMap == kMapElu1 || part == 1) {
#pragma unroll
      for (int c = 0; c < P; ++c) top = largest(f[c], top);
    }
    write_pieces<F>(top, [&](auto inf) {
#pragma unroll
      for (int c = 0; c < P; ++c)
        F::template put<decltype(inf)::value>(mine + buffer * kBuffer + c * F::kTileBytes, row & 15, L.ch, f[c]);
    });
  };
  bool next_live = row_at(begin + 2 * kRound);
#pragma unroll
  for (int i = 0; i < 2; ++i) live[i] = row_at(begin + i * kRound);
#pragma unroll
  for (int i = 0; i < 2; ++i) load(raw[i], begin + i * kRound, live[i]);
  stage(raw[0], live[0], 0);
  live[0] = next_live;
  load(raw[0], begin + 2 * kRound, live[0]);
  next_live = row_at(begin + 3 * kRound);
#pragma unroll 1
  for (int r0 = begin; r0 < end; r0 += 2 * kRound) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = r0 + j * kRound;  // the round that is added, from buffer j; the next one goes to 1 - j
      if (r < end) {
        __syncthreads();  // round r is staged; nobody reads the other buffer any more
        const auto advance = [&] {
          stage(raw[1 - j], live[1 - j], 1 - j);
          live[1 - j] = next_live;
          load(raw[1 - j], r + 3 * kRound, live[1 - j]);
          next_live = row_at(r + 4 * kRound);
        };
        const int* flags = live_halves + 4 * j + 2 * part;
        const bool any = __builtin_amdgcn_readfirstlane(flags[0] | flags[1]) != 0;
        if (part == 0) advance();
        if (any) {
          const unsigned char* at = smem + j * kBuffer;
          const Pieces l0 = F::rows_operand(at + left, L);
          const Pieces l1 = F::rows_operand(at + left + F::kTileBytes, L);
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const Pieces y = F::rows_operand(at + right + b * F::kTileBytes, L);
            acc[0][b].add(l0, y);
            acc[1][b].add(l1, y);
          }
        }
        if (part == 1) advance();
      }
    }
  }
  request();
  __syncthreads();  // the tiles are overwritten next
  // of the 2 x 2 blocks of a quadrant the first half of the workgroup completes the first row, the
  // second half the second; first half's sum + second half's sum
  out.p = p0 + part;
  out.q0 = q0;
  out.here = true;
  f32x4_t* meet = reinterpret_cast<f32x4_t*>(smem) + L.lane;  // [wave that reads][block][quad][lane]
  static_assert(16 * 4 * 64 * 16 <= Map::kTiles, "the sums meet in the tiles");
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      meet[(((L.wave ^ 4) * 2 + b) * 4 + g) * 64] = part == 0 ? acc[1][b].group(g) : acc[0][b].group(g);
  __syncthreads();
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    out.v[b].zero();
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4_t own = part == 0 ? acc[0][b].group(g) : acc[1][b].group(g);
      out.v[b].add_group(g, own + meet[((L.wave * 2 + b) * 4 + g) * 64]);
    }
  }
  __syncthreads();
}

template <class F, int P, int WAVES, bool SWAPPED, class Request>
__device__ __forceinline__ void state_walk(State<F, P>& out, const Buffers& X, const Buffers& Y, int stride,
                                           const uint8_t* __restrict__ m, int begin, int end, float eps,
                                           const Lane& L, Request&& request) {
  if constexpr (P == 4) walk_quadrants<F, SWAPPED>(out, X, Y, stride, m, begin, end, eps, L, request);
  else if constexpr (WAVES == 4) walk_private<F, SWAPPED>(out, X, Y, stride, m, begin, end, eps, L, request);
  else walk_shared<F, SWAPPED>(out, X, Y, stride, m, begin, end, eps, L, request);
}

// The wave's blocks of scale * state into a set of images, image (p, q) that of piece p of x against piece q
// of y: DIRECT, straight from the lanes (transposed images after a plain walk, natural ones after a swapped
// one), or the other ones, by way of the neighbouring lanes.
template <class F, int P, bool SWAPPED, bool DIRECT>
__device__ __forceinline__ void state_images(const State<F, P>& s, float scale, unsigned char* images, const Lane& L) {
  if (!s.here) return;
#pragma unroll
  for (int j = 0; j < State<F, P>::kBlocks; ++j) {
    const int index = SWAPPED ? P * (s.q0 + j) + s.p : P * s.p + s.q0 + j;
    quadrant_image<F, !DIRECT>([&](int g) { return s.v[j].group(g); }, scale, images + index * F::kImageBytes, L);
  }
}

// The wave's blocks (of a plain walk) into a row-major D x D array.
template <class F, int P>
__device__ __forceinline__ void state_rows(const State<F, P>& s, float* __restrict__ out, const Lane& L) {
  constexpr int D = P * F::D;
  if (!s.here) return;
#pragma unroll
  for (int j = 0; j < State<F, P>::kBlocks; ++j)
#pragma unroll
    for (int g = 0; g < F::Acc::kGroups; ++g) {
      const f32x4_t v = s.v[j].group(g);
      float* at = out + (s.p * F::D + F::Acc::group_row(g, L)) * D + (s.q0 + j) * F::D + F::Acc::group_col(g, L);
#pragma unroll
      for (int i = 0; i < 4; ++i) at[i * D] = v[i];
    }
}

// ---- apply ----------------------------------------------------------------------------------------------

// 1/r of the lane's row under the cosine map (0 for a row that does not take part), 1 under ELU + 1.
template <class F, int P>
__device__ __forceinline__ float own_factor(const OwnRaw<P>& t, float eps, bool live, const Lane& L) {
  if (F::kMap == kMapElu1) return 1.0f;
  float ss = 0.0f;
#pragma unroll
  for (int c = 0; c < P; ++c) {
    float f[2 * F::EPL];
    own_values<F, P>(t, c, f);
#pragma unroll
    for (int i = 0; i < 2 * F::EPL; ++i) ss += f[i] * f[i];
  }
  return inv_norm_or_zero(row_sum_groups(ss, L), eps, live);
}

// The rows as they enter a product whose result is multiplied by own_factor(): raw, or phi(x).
template <class F, int P>
__device__ __forceinline__ void own_mapped(const OwnRaw<P>& t, bool live, typename F::TileRows (&x)[P]) {
  if (F::kMap != kMapElu1) {
    own_rows<F, P, false>(t, x);
    return;
  }
  float top = 0.0f;  // (phi(x) is infinite where x is)
#pragma unroll
  for (int c = 0; c < P; ++c) top = F::largest_raw(t.r[c][0], F::largest_raw(t.r[c][1], top));
  write_pieces<F>(top, [&](auto inf) {
#pragma unroll
    for (int c = 0; c < P; ++c) {
      float f[2 * F::EPL];
      own_values<F, P>(t, c, f);
#pragma unroll
      for (int i = 0; i < 2 * F::EPL; ++i) f[i] = elu1_or_zero(f[i], live);
      x[c].template set<decltype(inf)::value>(f);
    }
  });
}

// out = sum_c X[c] W(first + c * step)
template <class F, int P>
__device__ __forceinline__ void product(const typename F::TileRows (&X)[P], const unsigned char* images, int first,
                                        int step, const Lane& L, float (&out)[2 * F::EPL]) {
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
                                            const float (&o)[2 * F::EPL]) {
  if (row < end)
    store_product_row<F, kStoreStreamed>(out + c * kRowBytes, row, RowAddr{stride, kRowBytes}, L, o);
}

template <class F, int P>
__device__ __forceinline__ void store_zeros(unsigned char* out, int row, int end, int stride, const Lane& L) {
  float z[2 * F::EPL];
#pragma unroll
  for (int i = 0; i < 2 * F::EPL; ++i) z[i] = 0.0f;
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
    float o[2 * F::EPL];
    product<F, P>(x, images, q, P, L, o);
#pragma unroll
    for (int i = 0; i < 2 * F::EPL; ++i) o[i] *= inv;
    store_piece<F, P>(out, q, row, end, stride, L, o);
  }
}

// One tile of out = J (y rows) M^T, J the derivative of the map at the x rows (contraction over the
// columns of M; `images`: the natural ones).  Returns (mapped x) . (y M^T) of the lane's row.
// `y_used` may take the registers of y for the next tile.
template <class F, int P, class Used>
__device__ __forceinline__ float projected_tile(const OwnRaw<P>& x, const OwnRaw<P>& y, bool live, float inv,
                                                const unsigned char* images, unsigned char* out, int row, int end,
                                                int stride, const Lane& L, bool want_dot, Used&& y_used) {
  float g[P][2 * F::EPL];
  {
    typename F::TileRows Y[P];
    own_rows<F, P, true>(y, Y);
    y_used();
#pragma unroll
    for (int p = 0; p < P; ++p) product<F, P>(Y, images, P * p, 1, L, g[p]);
  }
  float dot = 0.0f;
  if (F::kMap != kMapElu1 || want_dot) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      float f[2 * F::EPL];
      own_values<F, P>(x, p, f);
#pragma unroll
      for (int i = 0; i < 2 * F::EPL; ++i)
        dot += (F::kMap == kMapElu1 ? elu1_or_zero(f[i], live) : f[i] * inv) * g[p][i];
    }
    dot = row_sum_groups(dot, L);
  }
#pragma unroll
  for (int p = 0; p < P; ++p) {
    float f[2 * F::EPL];
    own_values<F, P>(x, p, f);
#pragma unroll
    for (int i = 0; i < 2 * F::EPL; ++i)
      g[p][i] = F::kMap == kMapElu1 ? g[p][i] * fminf(elu1(f[i]), 1.0f) : (g[p][i] - f[i] * inv * dot) * inv;
    store_piece<F, P>(out, p, row, end, stride, L, g[p]);
  }
  return dot;
}

struct Range {
  int begin, end, stride;
};

// The images afresh for every tile: left alone the compiler reads the operands of all of them once, ahead
// of the tile loop, into registers that it does not have.
__device__ __forceinline__ const unsigned char* afresh(const unsigned char* images) {
  int zero = 0;
  asm volatile("" : "+s"(zero));
  return images + zero;
}

__device__ __forceinline__ bool row_live(const uint8_t* keys, int row, int end) {
  return row < end && (keys == nullptr || keys[row] != 0);
}

// O, or dV alone.  `first`: the wave's first tile, already requested.
template <class F, int P, int WAVES>
__device__ __forceinline__ void apply_plain(const Buffers& X, const uint8_t* keys, const Range r, float eps,
                                            const unsigned char* images, unsigned char* out, const Lane& L,
                                            const OwnRaw<P>& first) {
  constexpr int kStep = WAVES * TR;
  const RowAddr addr{r.stride, P * kRowBytes};
  OwnRaw<P> next = first;
  bool next_live = row_live(keys, r.begin + L.wave * TR + L.i16, r.end);
#pragma unroll 1
  for (int row0 = r.begin + L.wave * TR; row0 < r.end; row0 += kStep) {
    const OwnRaw<P> cur = next;
    const unsigned char* set = afresh(images);
    const bool live = next_live;
    const int row = row0 + L.i16;
    next_live = row_live(keys, row + kStep, r.end);
    load_own<P>(next, L, X, addr, row0 + kStep, next_live);
    if (keys != nullptr && __builtin_amdgcn_ballot_w64(live) == 0) {
      store_zeros<F, P>(out, row, r.end, r.stride, L);
      continue;
    }
    plain_tile<F, P>(cur, live, own_factor<F, P>(cur, eps, live, L), set, out, row, r.end, r.stride, L);
  }
}

// dQ, or dK alone (natural images; returns this lane's share of sum_i x_i . (y_i M^T)), or dK and dV (BOTH: from both
// sets, K is read once).
template <class F, int P, int WAVES, bool BOTH>
__device__ __forceinline__ float apply_projected(const Buffers& X, const Buffers& Y, const uint8_t* keys,
                                                 const Range r, float eps, const unsigned char* images,
                                                 const unsigned char* transposed, unsigned char* out,
                                                 unsigned char* out_plain, const Lane& L,
                                                 const OwnRaw<P>& first_x, const OwnRaw<P>& first_y,
                                                 bool want_dot) {
  constexpr int kStep = WAVES * TR;
  const RowAddr addr{r.stride, P * kRowBytes};
  float dots = 0.0f;
  OwnRaw<P> nx = first_x, y = first_y;
  bool next_live = row_live(keys, r.begin + L.wave * TR + L.i16, r.end);
#pragma unroll 1
  for (int row0 = r.begin + L.wave * TR; row0 < r.end; row0 += kStep) {
    const OwnRaw<P> x = nx;
    const bool live = next_live;
    next_live = row_live(keys, row0 + kStep + L.i16, r.end);
    load_own<P>(nx, L, X, addr, row0 + kStep, next_live);
    const auto next_y = [&] { load_own<P>(y, L, Y, addr, row0 + kStep, next_live); };
    const OwnRaw<P> cur_y = y;
    if (P == 2) next_y();  // (four pieces: once the registers are free)
    const int row = row0 + L.i16;
    if (keys != nullptr && __builtin_amdgcn_ballot_w64(live) == 0) {
      if (P == 4) next_y();
      store_zeros<F, P>(out, row, r.end, r.stride, L);
      if (BOTH) store_zeros<F, P>(out_plain, row, r.end, r.stride, L);
      continue;
    }
    const float inv = own_factor<F, P>(x, eps, live, L);
    if (BOTH) plain_tile<F, P>(x, live, inv, afresh(transposed), out_plain, row, r.end, r.stride, L);
    const float dot = projected_tile<F, P>(x, cur_y, live, inv, afresh(images), out, row, r.end, r.stride, L, want_dot, [&] {
      if (P == 4) next_y();
    });
    if (L.g16 == 0) dots += dot;
  }
  return dots;
}

// ---- one launch per direction ------------------------------------------------------------------------------

template <class F, int P, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 4 ? 3 : 2) void fused_fwd_kernel(const Args a) {
  constexpr int D = P * F::D;
  const Lane L;
  const int bh = blockIdx.x, N = a.N, stride = a.st.row.stride;
  const size_t base = a.st.slice_base(bh, a.H);
  const uint8_t* keys = a.keys_of(bh);
  State<F, P> s;
  const Buffers Q(a.Q + base, N, a.st.row);
  OwnRaw<P> first;
  {
    const Buffers K(a.K + base, N, a.st.row), V(a.V + base, N, a.st.row);
    state_walk<F, P, WAVES, false>(s, K, V, stride, keys, walk_begin<P>(keys, N, L), N, a.eps, L, [&] {
      load_own<P>(first, L, Q, a.st.row, L.wave * TR, L.wave * TR + L.i16 < N);
    });
  }
  state_images<F, P, false, true>(s, a.scale_of(bh), smem, L);
  if (a.kept != nullptr) state_rows<F, P>(s, a.kept + static_cast<size_t>(bh) * D * D, L);
  __syncthreads();
  apply_plain<F, P, WAVES>(Q, nullptr, Range{0, N, stride}, a.eps, smem, a.O + base, L, first);
}

template <class F, int P, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 4 ? 3 : 2) void fused_bwd_kernel(const Args a) {
  typedef Lds<F, P, WAVES> Map;
  const Lane L;
  // workgroups go to the XCDs round-robin: the two roles of a slice are eight apart, on one XCD
  const int bh = (blockIdx.x >> 4) * 8 + (blockIdx.x & 7);
  const bool second = ((blockIdx.x >> 3) & 1) != 0;  // dS, dV, dK
  if (bh >= a.slices) return;
  const int N = a.N, stride = a.st.row.stride;
  const size_t base = a.st.slice_base(bh, a.H);
  const uint8_t* keys = a.keys_of(bh);
  const float scale = a.scale_of(bh);
  const Buffers Q(a.Q + base, N, a.st.row), K(a.K + base, N, a.st.row);
  const Buffers V(a.V + base, N, a.st.row), dO(a.dO + base, N, a.st.row);
  const Range all{0, N, stride};
  const int row0 = L.wave * TR;
  State<F, P> s;
  OwnRaw<P> fx, fy;
  if (!second) {
    state_walk<F, P, WAVES, true>(s, K, V, stride, keys, walk_begin<P>(keys, N, L), N, a.eps, L, [&] {
      load_own<P>(fx, L, Q, a.st.row, row0, row0 + L.i16 < N);
      load_own<P>(fy, L, dO, a.st.row, row0, row0 + L.i16 < N);
    });
    state_images<F, P, true, true>(s, scale, smem, L);
    __syncthreads();
    float dots = apply_projected<F, P, WAVES, false>(Q, dO, nullptr, all, a.eps, smem, nullptr, a.dQ + base, nullptr,
                                                     L, fx, fy, a.dlog != nullptr);
    if (a.dlog != nullptr) {  // sum_i dO_i . O_i = sum_i qhat_i . (scale dO_i S^T), in a fixed order
      float* partial = reinterpret_cast<float*>(smem + Map::kWords);
      dots = wave_sum(dots);
      if (L.lane == 0) partial[L.wave] = dots;
      __syncthreads();
      if (threadIdx.x == 0) {
        float sum = 0.0f;
        for (int w = 0; w < WAVES; ++w) sum += partial[w];
        a.dlog[bh] = sum;
      }
    }
    return;
  }
  const bool live = row_live(keys, row0 + L.i16, N);
  state_walk<F, P, WAVES, false>(s, Q, dO, stride, nullptr, 0, N, a.eps, L, [&] {
    load_own<P>(fx, L, K, a.st.row, row0, live);
    if (P == 2) load_own<P>(fy, L, V, a.st.row, row0, live);
  });
  state_images<F, P, false, true>(s, scale, smem, L);
  if constexpr (P == 2) {
    state_images<F, P, false, false>(s, scale, smem + Map::kSet, L);
    __syncthreads();
    apply_projected<F, P, WAVES, true>(K, V, keys, all, a.eps, smem + Map::kSet, smem, a.dK + base, a.dV + base, L,
                                       fx, fy, false);
  } else {
    __syncthreads();
    apply_plain<F, P, WAVES>(K, keys, all, a.eps, smem, a.dV + base, L, fx);
    load_own<P>(fx, L, K, a.st.row, row0, live);
    load_own<P>(fy, L, V, a.st.row, row0, live);
    __syncthreads();  // nobody reads the transposed images any more
    state_images<F, P, false, false>(s, scale, smem, L);
    __syncthreads();
    apply_projected<F, P, WAVES, false>(K, V, keys, all, a.eps, smem, nullptr, a.dK + base, nullptr, L, fx, fy, false);
  }
}

// ---- three launches --------------------------------------------------------------------------------------------

// grid (slices * splits, 1 or 2); blockIdx.y == 1 reduces (Q, dO) instead of (K, V) under the key mask.
// Partial states: row-major D x D floats per workgroup, the second kind behind all of the first.
template <class F, int P, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 4 ? 3 : 2) void state_kernel(const Args a, float* __restrict__ ws) {
  constexpr int D = P * F::D;
  const Lane L;
  const int split = blockIdx.x % a.splits, bh = blockIdx.x / a.splits;
  const bool second = blockIdx.y == 1;
  const size_t base = a.st.slice_base(bh, a.H);
  const Buffers X((second ? a.Q : a.K) + base, a.N, a.st.row), Y((second ? a.dO : a.V) + base, a.N, a.st.row);
  const int begin = split * a.rows_per_split;
  const int end = a.N < begin + a.rows_per_split ? a.N : begin + a.rows_per_split;
  State<F, P> s;
  state_walk<F, P, WAVES, false>(s, X, Y, a.st.row.stride, second ? nullptr : a.keys_of(bh), begin, end, a.eps, L,
                                  [] {});
  state_rows<F, P>(s, ws + (static_cast<size_t>(blockIdx.y) * gridDim.x + blockIdx.x) * D * D, L);
}

// The images of scale * M (M: a complete state in global memory, row-major D x D): block (p, q) at
// P p + q, natural op[m][n] or transposed op[n][m] = M[p F::D + m][q F::D + n].
template <class F, int P, int WAVES, bool TRANSPOSED>
__device__ __forceinline__ void build_images(const float* __restrict__ M, float scale, unsigned char* images) {
  constexpr int D = P * F::D, kThreads = 64 * WAVES, kPairs = D * D / 2;
  constexpr int kBatch = kPairs / kThreads < 8 ? kPairs / kThreads : 8;  // whose loads travel together
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
    write_pieces<F>(largest(v0, largest(v1)) * scale, [&](auto inf) {
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const int e = e0 + j * kThreads;
        const int m = TRANSPOSED ? 2 * (e / D) : e / (D / 2);
        const int n = TRANSPOSED ? e % D : 2 * (e % (D / 2));
        unsigned char* image = images + (P * (m / F::D) + n / F::D) * F::kImageBytes;
        if (TRANSPOSED) F::template write_image_pair<decltype(inf)::value>(image, n % F::D, m % F::D, v0[j] * scale, v1[j] * scale);
        else F::template write_image_pair<decltype(inf)::value>(image, m % F::D, n % F::D, v0[j] * scale, v1[j] * scale);
      }
    });
  }
}

template <class F, int P, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 4 ? 3 : 2) void apply_fwd_kernel(const Args a) {
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
  build_images<F, P, WAVES, true>(a.states + static_cast<size_t>(bh) * D * D, a.scale_of(bh), smem);
  __syncthreads();
  apply_plain<F, P, WAVES>(Q, nullptr, Range{begin, end, a.st.row.stride}, a.eps, smem, a.O + base, L, first);
}

// blockIdx.y: 0 dQ, 1 dV, 2 dK
template <class F, int P, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 4 ? 3 : 2) void apply_bwd_kernel(const Args a) {
  constexpr int D = P * F::D;
  const Lane L;
  const int split = blockIdx.x % a.splits, bh = blockIdx.x / a.splits, role = blockIdx.y;
  const size_t base = a.st.slice_base(bh, a.H);
  const int begin = split * a.rows_per_split;
  const int end = a.N < begin + a.rows_per_split ? a.N : begin + a.rows_per_split;
  const int row0 = begin + L.wave * TR;
  const Range rows{begin, end, a.st.row.stride};
  const uint8_t* keys = role == 0 ? nullptr : a.keys_of(bh);
  const Buffers X((role == 0 ? a.Q : a.K) + base, a.N, a.st.row), Y((role == 0 ? a.dO : a.V) + base, a.N, a.st.row);
  const float* M = (role == 0 ? a.states : a.dstates) + static_cast<size_t>(bh) * D * D;
  const bool live = row_live(keys, row0 + L.i16, end);
  OwnRaw<P> fx, fy;
  load_own<P>(fx, L, X, a.st.row, row0, live);
  if (role == 1) {
    build_images<F, P, WAVES, true>(M, a.scale_of(bh), smem);
    __syncthreads();
    apply_plain<F, P, WAVES>(X, keys, rows, a.eps, smem, a.dV + base, L, fx);
  } else {
    load_own<P>(fy, L, Y, a.st.row, row0, live);
    build_images<F, P, WAVES, false>(M, a.scale_of(bh), smem);
    __syncthreads();
    apply_projected<F, P, WAVES, false>(X, Y, keys, rows, a.eps, smem, nullptr, (role == 0 ? a.dQ : a.dK) + base,
                                        nullptr, L, fx, fy, false);
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
  const long long e = p.elem_bytes();
  a.st = Strides{p.stride_batch * e, p.stride_head * e,
                 RowAddr{static_cast<int>(p.stride_row * e), static_cast<int>(p.D * e)}};
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

template <class F, int P, int WAVES>
hipError_t run(Kind kind, const Problem& p, const Args& a, bool bwd) {
  constexpr int threads = 64 * WAVES, lds = Lds<F, P, WAVES>::kBytes;
  static_assert(lds <= 160 * 1024 / (WAVES == 4 ? 3 : 1), "three workgroups per compute unit, or one");
  const unsigned slices = static_cast<unsigned>(a.slices);
  if (kind == kFused)
    return bwd ? launch(fused_bwd_kernel<F, P, WAVES>, dim3((slices + 7) / 8 * 16), threads, lds, p, a)
               : launch(fused_fwd_kernel<F, P, WAVES>, dim3(slices), threads, lds, p, a);
  const unsigned blocks = slices * a.splits;
  if (kind == kStates)
    return launch(state_kernel<F, P, WAVES>, dim3(blocks, bwd ? 2 : 1), threads, lds, p, a, p.workspace);
  return bwd ? launch(apply_bwd_kernel<F, P, WAVES>, dim3(blocks, 3), threads, lds, p, a)
             : launch(apply_fwd_kernel<F, P, WAVES>, dim3(blocks), threads, lds, p, a);
}

template <bool ELU>
hipError_t choose(Kind kind, const Problem& p, const Args& a, bool bwd) {
  typedef typename std::conditional<ELU, WithElu1<F32x32>, F32x32>::type F;
  typedef typename std::conditional<ELU, WithElu1<F32x32Apart>, F32x32Apart>::type Apart;
  // (d_h = 128: apart at every length, 8 x 200 rows 21.5 / 35.4, plain 21.8 / 36.0;  128 x 200 23.7 / 38.9, 24.0 / 39.3)
  if (p.D == 128) return run<Apart, 4, 8>(kind, p, a, bwd);
  // Eight waves where there is a compute unit for every workgroup (forward / backward, us, four and
  // eight: 128 slices x 200 rows 15.8 / 20.3, 12.9 / 17.5; 8 slices 13.5 / 18.3, 10.5 / 15.1).
  constexpr long kUnits = 256;
  const bool few = static_cast<long>(a.slices) * a.splits * (bwd ? 2 : 1) <= kUnits;
  // Sequences, or parts of them, of more than 256 rows are summed apart.  (Shorter ones have no need, and it costs time: 4
  // slices x 200 rows 10.6 / 14.8 plain, 11.0 / 15.2.  Nor do they where there are more slices than compute units.)
  if (a.rows_per_split <= 256) return few ? run<F, 2, 8>(kind, p, a, bwd) : run<F, 2, 4>(kind, p, a, bwd);
  if (few) return run<Apart, 2, 8>(kind, p, a, bwd);
  return a.slices <= kUnits ? run<Apart, 2, 4>(kind, p, a, bwd) : run<F, 2, 4>(kind, p, a, bwd);
}

hipError_t dispatch(Kind kind, const Problem& p, const Args& a, bool bwd) {
  return p.feature_map == kMapElu1 ? choose<true>(kind, p, a, bwd) : choose<false>(kind, p, a, bwd);
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
