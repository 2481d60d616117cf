// skew_kernels.hip -- gfx950 kernels of one SkewAdam step (Sec. 3, Eq. 1, Alg. 1).
//
// A step is a short sequence of stream-ordered launches over device-resident work-item
// tables; each launch covers every tensor of the table (e.g. all experts of a layer):
//   p1z   factored matrices up to 16384 columns (row-band pass): R_i, partial column sums
//         of g^2 and of (s x)^2 / R_i, the floored sum of U_hat^2 and bounds, in one read of G
//   p1    wider factored matrices: per tile, partial row and column sums of g^2 (Eq. 1)
//   fold  factored tensors: C (and for wide ones R) EMA (Eq. 1), 1/sqrt(R_i), c'_j and
//         the row-band tensors' sum of U_hat^2 above the floor
//   p2    exact-second-moment tensors and wide factored ones: per tile, sum of squares of
//         the unclipped update (Alg. 1)
//   clip  per tensor: the clip factor k, and whether its rounding needs the exact pass
//         (the slices of stacked tensors first, one wave each, in a launch of their own)
//   p2x   re-runs of the sum for the tensors the clip stage left undecided (the exact floor
//         split, then the oracle's float sequence); clip again
//   p3    every tensor: momentum / exact-v update, weight update, dithered bf16
//         write-back (Sec. 3 "Update clipping and low-precision updates")
// Reductions are deterministic (fixed-order partials; no float atomics), so two
// runs on the same inputs produce identical bits.
//
// Tile (p1, p2, p3): tr rows x (512*cw) columns. A work-group is 4 wave64; lane l covers 8
// consecutive columns (one 16-byte bf16 load) in each 512-column chunk.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <type_traits>

#include "skew_internal.h"

namespace skew {
namespace {

// Tensor pointers come from the device-resident table, so the compiler cannot infer
// their address space; these accessors make every data access a global (not flat) one.
template <class T>
__device__ __forceinline__ T ldg(const T *p) {
  return *(const __attribute__((address_space(1))) T *)p;
}
template <class T>
__device__ __forceinline__ void stg(T *p, T v) {
  *(__attribute__((address_space(1))) T *)p = v;
}
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ldg(const float4 *p) {
  const f32x4_t v = ldg(reinterpret_cast<const f32x4_t *>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void stg(float4 *p, float4 v) {
  const f32x4_t u = {v.x, v.y, v.z, v.w};
  stg(reinterpret_cast<f32x4_t *>(p), u);
}
// Non-temporal 16-byte loads and stores, for the bf16 gradient and weight rows that the update
// pass streams through once (a hint to the caches not to keep them). Together they took the
// 6.78B update pass from 8.07 to 7.65 ms; loads alone (8.23) or stores alone (8.12) did not,
// and on the fp32 momentum the hint costs time (the expert-momentum variant: 18.1 -> 19.2 ms).
template <class V>
__device__ __forceinline__ V ldg_nt(const V *p) {
  return __builtin_nontemporal_load((const __attribute__((address_space(1))) V *)p);
}
template <class V>
__device__ __forceinline__ void stg_nt(V *p, V v) {
  __builtin_nontemporal_store(v, (__attribute__((address_space(1))) V *)p);
}
__device__ __forceinline__ uint4 ldg_nt(const uint4 *p) {
  const u32x4_t v = ldg_nt(reinterpret_cast<const u32x4_t *>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void stg_nt(uint4 *p, uint4 v) {
  const u32x4_t u = {v.x, v.y, v.z, v.w};
  stg_nt(reinterpret_cast<u32x4_t *>(p), u);
}

__device__ __forceinline__ float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }
// max(a, b) that returns `a` when it is NaN (b is a finite constant): NaN propagates.
__device__ __forceinline__ float max_nan(float a, float b) { return (a < b) ? b : a; }

__device__ __forceinline__ void unpack8(const uint4 &u, float *o) {
  o[0] = bf_lo(u.x); o[1] = bf_hi(u.x);
  o[2] = bf_lo(u.y); o[3] = bf_hi(u.y);
  o[4] = bf_lo(u.z); o[5] = bf_hi(u.z);
  o[6] = bf_lo(u.w); o[7] = bf_hi(u.w);
}

// 8 momentum values at a 32-byte aligned position
__device__ __forceinline__ void load_m8(const float *p, float *o) {
  const float4 a = ldg(reinterpret_cast<const float4 *>(p));
  const float4 b = ldg(reinterpret_cast<const float4 *>(p + 4));
  o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}
__device__ __forceinline__ void store_m8(float *p, const float *v) {
  stg(reinterpret_cast<float4 *>(p), make_float4(v[0], v[1], v[2], v[3]));
  stg(reinterpret_cast<float4 *>(p + 4), make_float4(v[4], v[5], v[6], v[7]));
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// two floats -> two bf16, round to nearest even, packed low|high
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// SplitMix64 output function (Steele, Lea, Flood, OOPSLA 2014).
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
// MurmurHash3 32-bit finalizer (public domain).
__device__ __forceinline__ uint32_t fmix32(uint32_t h) {
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  h *= 0xC2B2AE35u;
  h ^= h >> 16;
  return h;
}

// Counter-based dither source: one 32-bit hash per element pair p = idx >> 1,
// keyed by (seed, step, tensor id). Element 2p takes the low 16 bits, 2p+1 the high.
struct Dither {
  uint32_t klo, khi, inner0;
  __device__ __forceinline__ Dither(uint64_t seed, int64_t step, uint64_t id) {
    const uint64_t k = mix64(mix64(mix64(seed) ^ (uint64_t)step) ^ id);
    klo = (uint32_t)k;
    khi = (uint32_t)(k >> 32);
    inner0 = fmix32(khi);
  }
  // the hash input of pair p before the final mix: pair(p) = fmix32(pair_base(p))
  __device__ __forceinline__ uint32_t pair_base(uint64_t p) const {
    const uint32_t ph = (uint32_t)(p >> 32);
    const uint32_t inner = (ph == 0u) ? inner0 : fmix32(ph ^ khi);
    return (uint32_t)p ^ klo ^ inner;
  }
  __device__ __forceinline__ uint32_t pair(uint64_t p) const { return fmix32(pair_base(p)); }
};

// e * 2^-24 with e = 2*u16 + 1 - 2^16 = u16 * 2^-23 + (1 - 2^16) * 2^-24: a multiple of
// 2^-24 below 2^-8 in magnitude, so the fma is exact (u16 converts exactly)
__device__ __forceinline__ float dither_u16(uint32_t u) { return fmaf((float)u, 0x1p-23f, -65535.0f * 0x1p-24f); }
__device__ __forceinline__ float dither_lo(uint32_t h) { return dither_u16(h & 0xFFFFu); }
__device__ __forceinline__ float dither_hi(uint32_t h) { return dither_u16(h >> 16); }

// Dither values of 8 elements from index idx on (any parity; `wide`: pair indices may pass 32 bits,
// else the pairs share their high word). An odd start takes the high half of its first pair, so
// the half-words of 5 pairs are shifted by one.
__device__ __forceinline__ void dither8(const Dither &dz, uint64_t idx, bool wide, float *d) {
  const uint64_t p0 = idx >> 1;
  const bool odd = (idx & 1u) != 0;
  uint32_t h[5];
#pragma unroll
  for (int e = 0; e < 5; e++) {
    if (e == 4 && !odd) {
      h[e] = 0u;
      continue;
    }
    h[e] = wide ? dz.pair(p0 + e) : fmix32(((uint32_t)p0 + (uint32_t)e) ^ dz.klo ^ dz.inner0);
  }
#pragma unroll
  for (int e = 0; e < 4; e++) {
    const uint32_t w = odd ? __builtin_amdgcn_alignbit(h[e + 1], h[e], 16) : h[e];
    d[2 * e] = dither_lo(w);
    d[2 * e + 1] = dither_hi(w);
  }
}

// The noise added before the cast is the product of two exact factors: e 2^-24 and |w|
// (ulp(w) taken as 2^-7 |w|, Sec. 3), or, in the exact-ulp mode, e 2^-24 and 2^7 times the
// bf16 ulp of w. That ulp is 2^(E - 134) for biased exponent E >= 1 and 2^-133 among the
// subnormals, so 2^7 ulp is the float whose exponent field is E clamped to [1, 254] (an
// infinite or NaN w keeps a finite factor; its update is infinite or NaN already)
__device__ __forceinline__ float bf16_ulp128(float w) {
  const uint32_t b = __float_as_uint(w) & 0x7F800000u;
  return __uint_as_float(min(max(b, 0x00800000u), 0x7F000000u));
}
__device__ __forceinline__ float dither_mul(float w, bool xu) { return xu ? bf16_ulp128(w) : fabsf(w); }

// Butterfly reductions over one wave64: every lane ends with the same value (each step
// adds two equal-order partials, and IEEE addition is commutative), so the result is
// deterministic.
__device__ __forceinline__ double wave_sum_d(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ __forceinline__ double wave_max_d(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o, 64));
  return x;
}
__device__ __forceinline__ float wave_min_f(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fminf(x, __shfl_xor(x, o, 64));
  return x;
}
__device__ __forceinline__ float wave_max_f(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}
__device__ __forceinline__ int wave_or(int x) { return __any(x != 0) ? 1 : 0; }

// Work-group reductions of NW waves through sh[NW] (every thread gets the result; the
// per-wave results are combined in wave order).
template <int NW>
__device__ __forceinline__ double wg_sum_w(double x, double *sh) {
  x = wave_sum_d(x);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = x;
  __syncthreads();
  double r = 0.0;
#pragma unroll
  for (int w = 0; w < NW; w++) r += sh[w];
  __syncthreads();
  return r;
}
// fixed-order sum over a work-group of kThreads (every thread gets the total)
__device__ __forceinline__ double block_sum(double x, double *sh) { return wg_sum_w<kWaves>(x, sh); }

// A tile is one row band (rows band, band + ntr, band + 2 ntr, ...: interleaved, so that
// the work-groups running at the same time on one tensor read neighbouring rows) times
// one column strip of 512*cw columns.
struct Tile {
  int64_t nr, c0, stride;   // local rows, first column, row stride between local rows
  int band, strip;
  __device__ __forceinline__ int64_t row(int64_t lr) const { return band + lr * stride; }
};
__device__ __forceinline__ Tile tile_of(const DevTensor &t, int tile) {
  Tile g;
  g.band = tile / t.ntc;
  g.strip = tile - g.band * t.ntc;
  g.stride = t.ntr;
  g.nr = (t.n - g.band + t.ntr - 1) / t.ntr;
  g.c0 = (int64_t)g.strip * kChunk * t.cw;
  return g;
}

// Wave -> (chunk, row) map inside a tile: the cw chunks of a row go to cw adjacent waves,
// so one work-group iteration reads kWaves / cw whole tile rows (up to 4 KB contiguous),
// and every wave keeps the same 512 columns for the whole tile.
struct WaveMap {
  int wq, wr, rpi, lane;
  int64_t col;   // first of the lane's 8 columns
  __device__ __forceinline__ WaveMap(const DevTensor &t, const Tile &tl) {
    const int wave = threadIdx.x >> 6;
    lane = threadIdx.x & 63;
    wq = wave % t.cw;
    wr = wave / t.cw;
    rpi = kWaves / t.cw;
    col = tl.c0 + (int64_t)wq * kChunk + lane * 8;
  }
};

// Rows at most this far apart are packed: 64 rows' offsets stay below 2^31 bytes
constexpr int64_t kPackLd = (int64_t(1) << 31) / 64 / 4;

// The update pass's map: a wave keeps its chunk of 512 columns for the whole tile, and where the
// chunk holds only `g` of the 64 groups of 8 columns (a narrow matrix, or the end of a row) its
// lanes take 64 / g rows at a time, so that a 7-column remainder does not cost as much as a whole
// chunk (update pass over 3.65e8 elements in rows of 1031 columns: 718 -> 570 us; 2.6e8 in rows of
// 256: 422 -> 290 us). The rows of a tile are blocks of that many rows, interleaved with the other
// bands'. Chunks of more than 32 groups take one row, with the offsets of a lane's row left out.
struct LaneMap {
  int64_t c0;            // the wave's first column (uniform)
  int64_t row, step;     // first row of the wave's first block of rows, and the step to its next (uniform)
  int sub;               // the lane's row within a block
  int col;               // its first column from c0 on (negative: see `over`)
  int over;              // its columns past the row's end; col moves back by as many (not in rows of < 8)
  bool idle;
  // whether the wave's chunk is narrow enough for two rows or more (uniform)
  static __device__ __forceinline__ bool packs(const DevTensor &t, const Tile &tl) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    return t.m - tl.c0 - (int64_t)(wave % t.cw) * kChunk <= kChunk / 2 && t.ld <= kPackLd;
  }
  __device__ __forceinline__ LaneMap(const DevTensor &t, const Tile &tl, bool pack) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wq = wave % t.cw, wr = wave / t.cw, rpi = kWaves / t.cw;
    c0 = tl.c0 + (int64_t)wq * kChunk;
    const int64_t left = t.m - c0;
    int g = 64, rpw = 1;
    if (pack && left > 0 && left <= kChunk / 2) {
      g = ((int)left + 7) >> 3;
      rpw = 64 / g;
    }
    sub = pack ? lane / g : 0;
    const int gi = lane - sub * g;
    row = (tl.band + (int64_t)wr * tl.stride) * rpw;
    step = (int64_t)rpi * tl.stride * rpw;
    idle = gi * 8 >= left || sub >= rpw;
    over = gi * 8 + 8 > left ? gi * 8 + 8 - (int)left : 0;
    col = gi * 8 - (t.m < 8 ? 0 : over);
  }
};

__device__ __forceinline__ uint4 to_uint4(const u32x4_t &v) { return make_uint4(v.x, v.y, v.z, v.w); }
// v shifted down by sh elements (0..7), zeros entering at the top: of 8 packed bf16 values,
// and of 8 floats in two halves
__device__ __forceinline__ void shift_down(u32x4_t &v, int sh) {
  const u32x4_t z4 = {v.z, v.w, 0u, 0u};
  if (sh & 4) v = z4;
  const u32x4_t z2 = {v.y, v.z, v.w, 0u};
  if (sh & 2) v = z2;
  const u32x4_t z1 = {__builtin_amdgcn_alignbit(v.y, v.x, 16), __builtin_amdgcn_alignbit(v.z, v.y, 16),
                      __builtin_amdgcn_alignbit(v.w, v.z, 16), v.w >> 16};
  if (sh & 1) v = z1;
}
__device__ __forceinline__ void shift_down(u32x4_t &a, u32x4_t &b, int sh) {
  const u32x4_t zero = {0u, 0u, 0u, 0u};
  if (sh & 4) {
    a = b;
    b = zero;
  }
  const u32x4_t a2 = {a.z, a.w, b.x, b.y}, b2 = {b.z, b.w, 0u, 0u};
  if (sh & 2) {
    a = a2;
    b = b2;
  }
  const u32x4_t a1 = {a.y, a.z, a.w, b.x}, b1 = {b.y, b.z, b.w, 0u};
  if (sh & 1) {
    a = a1;
    b = b1;
  }
}

// Rows at any position: 16-byte loads and stores of 8 bf16 values at a 2-byte position, and of 4
// floats at a 4-byte position (the hardware takes both; on aligned addresses at full speed)
// (types of their own, not template arguments, which would drop the alignment)
typedef unsigned u32x4_u2_t __attribute__((ext_vector_type(4), aligned(2)));
typedef float f32x4_u4_t __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ u32x4_t ldg_u(const uint16_t *p) {
  return *(const __attribute__((address_space(1))) u32x4_u2_t *)p;
}
// (non-temporal for the update pass, the gradient's last reader. In the passes before it the hint
// keeps G from the caches that the next one reads it from: 6.7e7 elements in rows of 20000 took the
// first pass, the update sums and the update 45, 67 and 107 us with it, 44, 65 and 98 without)
__device__ __forceinline__ u32x4_t ldg_u_nt(const uint16_t *p) {
  return __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4_u2_t *)p);
}
__device__ __forceinline__ u32x4_t ldg_u(const float *p) {
  return __builtin_bit_cast(u32x4_t, (f32x4_t)*(const __attribute__((address_space(1))) f32x4_u4_t *)p);
}
__device__ __forceinline__ void stg_u(uint16_t *p, u32x4_t v) {
  __builtin_nontemporal_store((u32x4_u2_t)v, (__attribute__((address_space(1))) u32x4_u2_t *)p);
}
__device__ __forceinline__ void stg_u(float *p, f32x4_t v) {
  *(__attribute__((address_space(1))) f32x4_u4_t *)p = v;
}

// The lane's 8 columns of a row of m: how many of them lie past its end (0 for all lanes but
// the last). Such a lane loads the row's last 8 elements and shifts the ones before its own
// out; a row of fewer than 8 is loaded element by element. Elements past the end read as 0.
struct Cols8 {
  int64_t col;
  int over;      // columns past the row's end
  bool narrow;   // m < 8
  __device__ __forceinline__ Cols8(int64_t m, int64_t c)
      : col(c), over(c + 8 > m ? (int)(c + 8 - m) : 0), narrow(m < 8) {}
  // relative to the first of the 8 elements that the lane loads
  __device__ __forceinline__ Cols8(int over_, bool narrow_) : col(narrow_ ? 0 : over_), over(over_), narrow(narrow_) {}
  __device__ __forceinline__ int count() const { return 8 - over; }
};
template <bool NT = false>
__device__ __forceinline__ u32x4_t load8(const uint16_t *row, const Cols8 &c) {
  u32x4_t v = {0u, 0u, 0u, 0u};
  if (c.narrow) {
#pragma unroll
    for (int e = 0; e < 8; e++)
      if (e < c.count()) v[e >> 1] |= (uint32_t)ldg(row + c.col + e) << (16 * (e & 1));
  } else {
    v = NT ? ldg_u_nt(row + c.col - c.over) : ldg_u(row + c.col - c.over);
    if (c.over) shift_down(v, c.over);
  }
  return v;
}
__device__ __forceinline__ void load8(const float *row, const Cols8 &c, float *o) {
  u32x4_t a = {0u, 0u, 0u, 0u}, b = a;
  if (c.narrow) {
#pragma unroll
    for (int e = 0; e < 8; e++)
      if (e < c.count()) (e < 4 ? a : b)[e & 3] = __float_as_uint(ldg(row + c.col + e));
  } else {
    a = ldg_u(row + c.col - c.over);
    b = ldg_u(row + c.col - c.over + 4);
    if (c.over) shift_down(a, b, c.over);
  }
#pragma unroll
  for (int e = 0; e < 4; e++) {
    o[e] = __uint_as_float(a[e]);
    o[4 + e] = __uint_as_float(b[e]);
  }
}
// (the row's last lane stores its count() first values as 4 + 2 + 1 of them)
__device__ __forceinline__ void store8(float *row, const Cols8 &c, const float *v) {
  if (c.over == 0) {
    stg_u(row + c.col, f32x4_t{v[0], v[1], v[2], v[3]});
    stg_u(row + c.col + 4, f32x4_t{v[4], v[5], v[6], v[7]});
  } else {
    const int n = c.count();
    float *p = row + c.col;
    const bool four = (n & 4) != 0;
    if (four) stg_u(p, f32x4_t{v[0], v[1], v[2], v[3]});
    p += n & 4;
    const float a = four ? v[4] : v[0], b = four ? v[5] : v[1];
    const float d = four ? v[6] : v[2];
    if (n & 2) {
      stg(p, a);
      stg(p + 1, b);
    }
    if (n & 1) stg(p + (n & 2), (n & 2) ? d : a);
  }
}
typedef unsigned u32x2_u2_t __attribute__((ext_vector_type(2), aligned(2)));
typedef unsigned u32_u2_t __attribute__((aligned(2)));
__device__ __forceinline__ void store8(uint16_t *row, const Cols8 &c, const uint4 &v) {
  if (c.over == 0) {
    stg_u(row + c.col, u32x4_t{v.x, v.y, v.z, v.w});
  } else {
    const int n = c.count();
    uint16_t *p = row + c.col;
    const bool four = (n & 4) != 0;
    if (four) *(__attribute__((address_space(1))) u32x2_u2_t *)p = u32x2_u2_t{v.x, v.y};
    p += n & 4;
    const uint32_t a = four ? v.z : v.x, b = four ? v.w : v.y;
    if (n & 2) *(__attribute__((address_space(1))) u32_u2_t *)p = a;
    if (n & 1) stg(p + (n & 2), (uint16_t)((n & 2) ? b : a));
  }
}
// 8 elements of a weight or gradient row, bf16 or float32 (float32 masters)
__device__ __forceinline__ void load_elems8(const uint16_t *base, int64_t row_off, const Cols8 &c, bool fp32, float *o) {
  if (fp32)
    load8(reinterpret_cast<const float *>(base) + row_off, c, o);
  else
    unpack8(to_uint4(load8(base + row_off, c)), o);
}

__device__ __forceinline__ void load_g8(const DevTensor &t, int64_t i, int64_t col, float *g) {
  if (col < t.m) {
    unpack8(to_uint4(load8(t.g + i * t.ld, Cols8(t.m, col))), g);
  } else {
#pragma unroll
    for (int e = 0; e < 8; e++) g[e] = 0.f;
  }
}

// --------------------------------------------------------------------------------------------
// p1: partial row / column sums of g^2 (Eq. 1: mean_c and mean_r of G (.) G).
// Squares of bf16 values are exact in double and the sums stay far from double
// rounding, so every partial is (nearly) the exact sum, independent of order.
// --------------------------------------------------------------------------------------------
constexpr int kRowSlots = (int)(kTileElems / kChunk);   // tile rows x chunks per row

__global__ __launch_bounds__(kThreads) void p1_kernel(const DevTensor *__restrict__ TT,
                                                      const Item *__restrict__ items) {
  __shared__ double colsh[kWaves][kChunk];
  __shared__ double rowsh[kRowSlots];
  const Item it = items[blockIdx.x];
  const DevTensor &t = TT[it.tensor];
  const Tile tl = tile_of(t, it.tile);
  const WaveMap wm(t, tl);
  const int cw = t.cw;

  double acc[8];
#pragma unroll
  for (int e = 0; e < 8; e++) acc[e] = 0.0;
  for (int64_t lr = wm.wr; lr < tl.nr; lr += 2 * wm.rpi) {
    const bool two = lr + wm.rpi < tl.nr;
    float ga[8], gb[8];
    load_g8(t, tl.row(lr), wm.col, ga);
    if (two) load_g8(t, tl.row(lr + wm.rpi), wm.col, gb);
    double ra = 0.0, rb = 0.0;
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const double x = (double)ga[e];
      ra = fma(x, x, ra);
      acc[e] = fma(x, x, acc[e]);
    }
    if (two) {
#pragma unroll
      for (int e = 0; e < 8; e++) {
        const double x = (double)gb[e];
        rb = fma(x, x, rb);
        acc[e] = fma(x, x, acc[e]);
      }
    }
    ra = wave_sum_d(ra);
    rb = wave_sum_d(rb);
    if (wm.lane == 0) {
      rowsh[lr * cw + wm.wq] = ra;
      if (two) rowsh[(lr + wm.rpi) * cw + wm.wq] = rb;
    }
  }
#pragma unroll
  for (int e = 0; e < 8; e++) colsh[threadIdx.x >> 6][wm.lane * 8 + e] = acc[e];
  __syncthreads();
  for (int r = threadIdx.x; r < (int)tl.nr; r += kThreads) {
    double s = 0.0;
    for (int q = 0; q < cw; q++) s += rowsh[r * cw + q];
    stg(t.rowpart + (int64_t)tl.strip * t.n + tl.row(r), s);
  }
  for (int c = threadIdx.x; c < kChunk * cw; c += kThreads) {
    const int q = c / kChunk, cc = c - q * kChunk;
    double s = 0.0;
    for (int w = q; w < kWaves; w += cw) s += colsh[w][cc];
    const int64_t col = tl.c0 + c;
    if (col < t.m) stg(t.colpart + (int64_t)tl.band * t.ldp + col, s);
  }
}

// --------------------------------------------------------------------------------------------
// Row-band pass: pass 1 of factored matrices up to 16384 columns (Eq. 1 and the update
// sum of Alg. 1 in one read of G).
//
// A work-group owns a band of whole rows, so R_i <- b2 R_i + a2 mean_j g_ij^2 is final as
// soon as row i is summed. With the row still at hand the work-group adds (s x_ij)^2 / R_i
// to a per-column sum z_j (x = g, or the new momentum on the backbone). Above the eps
// floor U_hat_ij^2 = (s x_ij)^2 / (R_i c'_j) up to the oracle's free roundings, so the
// tensor's sum of U_hat^2 is sum_j z_j / c'_j once the fold has c'_j = C_j / max(mean R,
// eps): no pass re-reads G for it. On the floor U_hat = RN(RN(s x) / sqrt(eps)) depends on
// x alone; its square is summed exactly as the oracle rounds it (Markstein's correctly
// rounded division). The clip stage takes whichever sum applies; the last step's
// regime decides which of the two this pass forms (a tensor that was clearly above the
// floor skips the floored sum, and the reverse).
//
// Roundings that repeat a pattern are replicated (RN(s x); the momentum fma), so the
// remaining difference from the oracle's sum is the free roundings of R_i c'_j, the
// square root and the quotient; the per-band maximum of (s x)^2 / R_i bounds their spread.
//
// Staging: every wave loads its own pieces of the next block of rows (bf16 gradient, and
// fp32 momentum on the backbone) straight into registers, by buffer loads of 16 bytes per
// lane, while it sums the current one: a whole block (up to 96 KiB a work-group) is in
// flight and no wave waits for another's loads. Rows may start at any 2-byte position (the
// hardware takes unaligned 16-byte loads); where the row is no multiple of 8 columns, the
// lane that holds its end loads the row's last 8 elements and shifts the ones before its
// own out.
//
// Layout: zcw 512-column chunks per row; a group of wpr = ceil(zcw / NSEG) waves shares a
// row, wave w of the group taking chunks w, w + wpr, ...; zrpi = 8 / wpr groups work on
// different rows. The column partials of the groups are added in group order through LDS.
// --------------------------------------------------------------------------------------------
// s_waitcnt immediate (gfx9 encoding): lgkmcnt(0) only
constexpr int kWaitLgkm0 = 0xC07F;

// bytes of a buffer's range (0 where a band has no block at all)
__device__ __forceinline__ int clamp_span(int64_t bytes) {
  return bytes <= 0 ? 0 : (bytes < 0x7FFFFFFF ? (int)bytes : 0x7FFFFFFF);
}

constexpr int kZRowSlots = kZMaxBlockRows * kZWaves;   // row partials of one block: [row][wave in group]
// column partials in LDS: 16 chunks of 512 columns (over the groups) at a time, element e of lane l's 8 columns at
// e * kColPad + l of its chunk (the writes of a wave and the reads of 64 consecutive columns
// both spread over all banks)
constexpr int kColPad = 72, kColChunks = 16;
constexpr int kZStats = 6;   // values of a band reduced over its work-group

// Cross-lane moves of doubles without LDS: DPP within 16-lane rows (quad permutes, half
// and full row mirrors) and the gfx950 lane-half swaps. Each reduction step adds two
// partials that both lanes of a pair add in the same order: results are deterministic.
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane i <-> 7 - i within each 8 lanes
constexpr int kDppMirror = 0x140;     // lane i <-> 15 - i within each 16 lanes
template <int CTRL>
__device__ __forceinline__ double dpp_d(double x) {
  // every lane reads a defined source lane under these patterns: no old value is needed
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
// a, b -> lanes < 32: a[l] + a[l + 32]; lanes >= 32: b[l - 32] + b[l]
__device__ __forceinline__ double swap32_add(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// a, b -> 16-lane rows 0, 2: a summed with the next row; rows 1, 3: b summed with the previous
__device__ __forceinline__ double swap16_add(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// Sums over the wave of RB values per lane (one per row), transposed: the lane halves and
// quarters exchange different rows first. Row b's total ends in lanes [b * 64/RB, (b + 1) * 64/RB).
template <int RB>
__device__ __forceinline__ double wave_sum_rows(const double (&v)[RB]) {
  const int lane = threadIdx.x & 63;
  double x;
  if constexpr (RB == 1) {
    const double w = swap32_add(v[0], v[0]);
    x = swap16_add(w, w);
  } else if constexpr (RB == 2) {
    const double w = swap32_add(v[0], v[1]);
    x = swap16_add(w, w);
  } else if constexpr (RB == 4) {
    x = swap16_add(swap32_add(v[0], v[2]), swap32_add(v[1], v[3]));
  } else {
    static_assert(RB == 8, "1, 2, 4 or 8 rows");
    const double u0 = swap16_add(swap32_add(v[0], v[4]), swap32_add(v[2], v[6]));
    const double u1 = swap16_add(swap32_add(v[1], v[5]), swap32_add(v[3], v[7]));
    const double a = u0 + dpp_d<kDppMirror>(u0), b = u1 + dpp_d<kDppMirror>(u1);
    x = (lane & 8) ? b : a;
  }
  x += dpp_d<kDppXor1>(x);
  x += dpp_d<kDppXor2>(x);
  x += dpp_d<kDppHalfMirror>(x);
  if constexpr (RB < 8) x += dpp_d<kDppMirror>(x);
  return x;
}
// exact (float)(x / d) for double x >= 0 and d > 0 with rd = RN(1 / d): the quotient is
// correctly rounded in double (Markstein) before the rounding to float
__device__ __forceinline__ float div_to_float(double x, double d, double rd) {
  const double q0 = x * rd;
  const double q = fma(fma(-q0, d, x), rd, q0);
  // an infinite (or NaN) sum is its own quotient; the correction would turn inf into NaN
  return (float)(__builtin_isfinite(q0) ? q : q0);
}
// 1 / x and 1 / sqrt(x) to about 2^-50 (hardware estimate and one Newton step)
__device__ __forceinline__ double rcp_d(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  return fma(y, fma(-x, y, 1.0), y);
}
__device__ __forceinline__ double rsq_d(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  return y * fma(-0.5 * x * y, y, 1.5);
}

// MODE 0: the whole pass; 1: the sums of g^2 alone (row sums to ainv; no momentum needed);
// 2: z, the floored sum and the band statistics of the scaled gradient, with R folded
// NARROW: rows of fewer than 8 columns, one column per lane in the first of its 8 places (no 16-byte
// load of the row's last 8 columns exists; the other places are zeros)
template <int NSEG, int RB, bool MOM, int MODE, bool NARROW = false>
__device__ __forceinline__ void p1z_body(const DevTensor &t, int band, const StepConsts &k, double *colbuf,
                                         double *rowsh, double *sh, float *rstash) {
  static_assert(MODE != 1 || !MOM, "the sums pass reads no momentum");
  static_assert(!NARROW || NSEG == 1, "a narrow row is one chunk");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t m = t.m, ld = t.ld;
  const int zcw = t.zcw;
  const int wpr = (zcw + NSEG - 1) / NSEG;   // waves per row
  const int grp = wave / wpr;
  const int wg = wave - grp * wpr;           // wave within the group
  const int rpi = t.zrpi;
  const int br = rpi * RB;                   // rows per block: RB per group
  const bool active = grp < rpi;
  const int grp_c = active ? grp : 0;        // idle waves read (and discard) group 0's rows
  int P = 1;                                 // wpr rounded up to a power of two
  while (P < wpr) P <<= 1;
  // The band's blocks of rows are band, band + nzb, ...: the work-groups that run at the same time
  // read neighbouring blocks, which spreads them over the memory channels (whole bands at power of
  // two distances do not)
  const int nzb = t.nzb;
  const int64_t nblk = ((t.n + br - 1) / br - band + nzb - 1) / nzb;
  auto first_row = [&](int64_t blk) { return (blk * nzb + band) * br; };
  const float sc = MOM ? k.s_m : k.s_0;
  const float deps = sqrtf(k.eps);                  // the oracle's D on the floor
  const float reps = (float)(1.0 / (double)deps);   // correctly rounded 1/D
  const double dm = (double)m, rdm = 1.0 / dm;
  // the sums this step forms (the clip stage's prediction from the last step)
  const int regime = __builtin_amdgcn_readfirstlane(ldg(&t.sc->regime));
  const bool want_z = regime != kRegimeFloor, want_y = regime != kRegimeAbove;

  // The lane's pieces: byte offsets from the block's first row, fixed for the whole band. Lanes
  // past the row's end take 2^31, beyond any block's range (the planner keeps a block's span
  // below 2^31), and rows past the matrix's end lie beyond the buffer's range by themselves: the
  // hardware returns zeros for both, so neither sweep masks anything. `tail` is the shift of the
  // lane whose 8 columns pass the row's end (its load moves back by as many columns).
  int chs[NSEG];
  constexpr bool VM = MOM && NSEG < 4;   // (rows over all waves: M's offsets are twice G's)
  uint32_t vo[RB][NSEG], vm[VM ? RB : 1][VM ? NSEG : 1];
  int tail = 0;
#pragma unroll
  for (int s = 0; s < NSEG; s++) {
    chs[s] = wg + s * wpr;
    const int64_t col = NARROW ? lane : (int64_t)chs[s] * kChunk + lane * 8;
    const bool ok = active && chs[s] < zcw && col < m;
    const int64_t over = !NARROW && col + 8 > m ? col + 8 - m : 0;
    if (ok && over) tail = (int)over;
#pragma unroll
    for (int b = 0; b < RB; b++) {
      const int64_t row = (int64_t)grp_c * RB + b;
      vo[b][s] = ok ? (uint32_t)((row * ld + col - over) * 2) : 0x80000000u;
      if constexpr (VM) vm[b][s] = ok ? (uint32_t)((row * m + col - over) * 4) : 0x80000000u;
    }
  }
  const bool ragged = !NARROW && (m & 7) != 0;

  double cacc[NSEG][8], zacc[NSEG][8];
#pragma unroll
  for (int s = 0; s < NSEG; s++)
#pragma unroll
    for (int e = 0; e < 8; e++) cacc[s][e] = zacc[s][e] = 0.0;
  double ysum = 0.0, ysum2 = 0.0, umax = 0.0;   // the floored sum in two chains
  double rs_l = 0.0;   // mode 1: the band's sum of g^2, kept by lane b * P of each group's first wave
  // mode 2: the gradient scale of the gradient-norm mode (elements enter as fl(c g))
  const float gc = MODE == 2 ? ldg(k.gscale) : 1.f;
  // a row with R_i == 0 but a nonzero sum (flagged by lane b * P of the group's first wave)
  int bad_l = 0;

  // the old R of the row whose fold the lane takes part in (lane b * P + w: row b of its group)
  const int rfold = grp_c * RB + ((lane / P) < RB ? (lane / P) : 0);
  auto issue_g = [&](int64_t blk, u32x4_t (&dst)[RB][NSEG], float &rold) {
    const int64_t rbase = first_row(blk);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(t.g + rbase * ld), (short)0, clamp_span((t.n - rbase) * ld * 2), 0x00020000);
#pragma unroll
    for (int b = 0; b < RB; b++)
#pragma unroll
      for (int s = 0; s < NSEG; s++) {
        if constexpr (NARROW)
          dst[b][s] = u32x4_t{(uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, vo[b][s], 0, 0), 0u, 0u, 0u};
        else
          dst[b][s] = __builtin_amdgcn_raw_buffer_load_b128(rs, vo[b][s], 0, 0);
      }
    if constexpr (MODE != 1) {
      const int64_t i = rbase + rfold;
      rold = ldg(t.R + (i < t.n ? i : t.n - 1));
    }
  };
  constexpr int MB = MOM ? RB : 1, MS = MOM ? NSEG : 1;
  auto issue_m = [&](int64_t blk, u32x4_t (&dst)[MB][MS][2]) {
    if constexpr (MOM) {
      const int64_t rbase = first_row(blk);
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void *)(t.M + rbase * m), (short)0, clamp_span((t.n - rbase) * m * 4), 0x00020000);
#pragma unroll
      for (int b = 0; b < RB; b++)
#pragma unroll
        for (int s = 0; s < NSEG; s++) {
          uint32_t o;
          if constexpr (VM) {
            o = vm[b][s];
          } else {
            o = vo[b][s];
            asm volatile("" : "+v"(o));   // formed here, not kept in a register of its own
            o = (o << 1) | (o & 0x80000000u);
          }
          if constexpr (NARROW) {
            dst[b][s][0] = u32x4_t{(uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, o, 0, 0), 0u, 0u, 0u};
            dst[b][s][1] = u32x4_t{0u, 0u, 0u, 0u};
          } else {
            dst[b][s][0] = __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0);
            dst[b][s][1] = __builtin_amdgcn_raw_buffer_load_b128(rs, o + 16u, 0, 0);
          }
        }
    }
  };
  // With one chunk per wave the momentum of the next block is in flight beside its gradient;
  // with more the registers hold one block of it, loaded at the start of its own step (it is
  // needed in the second sweep only)
  constexpr bool MDB = MOM && NSEG == 1;
  auto step = [&](int64_t blk, u32x4_t (&regc)[RB][NSEG], float rold, u32x4_t (&momc)[MB][MS][2],
                  u32x4_t (&regn)[RB][NSEG], float &rnold, u32x4_t (&momn)[MB][MS][2], auto zc, auto yc) {
    // the next block's loads go out first; the compiler waits for this block's registers
    // where they are first used
    if constexpr (MOM && !MDB) issue_m(blk, momc);
    if (blk + 1 < nblk) {
      issue_g(blk + 1, regn, rnold);
      if constexpr (MDB) issue_m(blk + 1, momn);
    }
    if (ragged) {   // the wave with the row's last chunk: the end's lane drops the elements before its own
#pragma unroll
      for (int s = 0; s < NSEG; s++)
        if (chs[s] == zcw - 1)
#pragma unroll
          for (int b = 0; b < RB; b++) {
            shift_down(regc[b][s], tail);
            if constexpr (MOM) shift_down(momc[b][s][0], momc[b][s][1], tail);
          }
    }
    const int64_t rbase = first_row(blk);
    double *slot = rowsh + (blk & 1) * kZRowSlots;   // [block row][wave in group]
    // row and column sums of g^2 (bf16 squares are exact in double); an idle wave's
    // accumulators are never used. Mode 2 has them from the first pass.
    if constexpr (MODE != 2) {
      double rp[RB];
#pragma unroll
      for (int b = 0; b < RB; b++) {
        double ra = 0.0, rb2 = 0.0;   // two chains per row
#pragma unroll
        for (int s = 0; s < NSEG; s++) {
          // one 8-element group at a time (the scheduler would otherwise convert every
          // staged element to double at once)
          __builtin_amdgcn_sched_barrier(0);
          float x[8];
          unpack8(to_uint4(regc[b][s]), x);
#pragma unroll
          for (int e = 0; e < 8; e++) {
            const double xd = (double)x[e];
            if (e & 1)
              rb2 = fma(xd, xd, rb2);
            else
              ra = fma(xd, xd, ra);
            cacc[s][e] = fma(xd, xd, cacc[s][e]);
          }
          // the column sums are formed here, not sunk towards the loop's end (which
          // would keep every converted element live across the block)
#pragma unroll
          for (int e = 0; e < 8; e++) asm volatile("" : "+v"(cacc[s][e]));
        }
        rp[b] = ra + rb2;
      }
      __builtin_amdgcn_sched_barrier(0);
      const double rsum = wave_sum_rows<RB>(rp);
      if (active && (lane & (64 / RB - 1)) == 0) slot[(grp * RB + lane / (64 / RB)) * kZWaves + wg] = rsum;
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
      __builtin_amdgcn_s_barrier();
    }
    // R_i after the EMA (Eq. 1) for the group's RB rows, lane-parallel: lane b * P + w
    // takes the partial of wave w of row b; after the segment sum lane b * P holds the row
    double winv_l = 0.0;
    {
      const int b = lane / P, w = lane - b * P;
      const int r = grp_c * RB + (b < RB ? b : 0);
      const int64_t i = rbase + r;
      const bool keeper = active && wg == 0 && b < RB && w == 0 && i < t.n;
      float R = rold;   // (mode 2: folded this step)
      double x = 0.0;
      if constexpr (MODE != 2) {
        x = (active && b < RB && w < wpr) ? slot[r * kZWaves + w] : 0.0;
        if (P >= 2) x += dpp_d<kDppXor1>(x);
        if (P >= 4) x += dpp_d<kDppXor2>(x);
        if (P >= 8) x += dpp_d<kDppHalfMirror>(x);
        if constexpr (MODE == 0) R = fmaf(k.a2, div_to_float(x, dm, rdm), __fmul_rn(k.b2, rold));
      }
      if constexpr (MODE == 1) {
        // the row's sum of g^2: R is folded once the gradient scale is known
        if (keeper) {
          stg(t.ainv + i, x);
          rs_l += x;
        }
      } else {
        const bool normal = R > 0.f && R < __builtin_inff();
        winv_l = (normal && i < t.n) ? rcp_d((double)R) : 0.0;   // (1/R is 0 for R = +inf)
        if (keeper) {
          // staged for the band's end: a global store here would hold up the next block's
          // wait for its staged rows until the store completes
          rstash[blk * br + r] = R;
          if (R != R || (MODE == 0 && !(R > 0.f) && x > 0.0)) bad_l = 1;
        }
      }
    }
    // z_j, the floored sum and the bound (the sums the prediction asks for)
    auto sweep2 = [&](auto zc, auto yc) {
      constexpr bool Z = decltype(zc)::value, Y = decltype(yc)::value;
#pragma unroll
      for (int b = 0; b < RB; b++) {
        const int src = b * P;
        const double winv = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(winv_l), src),
                                             __builtin_amdgcn_readlane(__double2loint(winv_l), src));
        float amax = 0.f;   // max |s x| over the lane's elements of the row
#pragma unroll
        for (int s = 0; s < NSEG; s++) {
          // one 8-element group at a time where registers are short
          if constexpr (MOM || NSEG > 2) __builtin_amdgcn_sched_barrier(0);
          float x[8];
          // the packed block is unpacked again here, from its own registers (not needed after
          // this sweep, so the empty asm may claim to change them: no copy is made); keeping
          // sweep 1's floats beside the next block's registers would spill
          asm volatile("" : "+v"(regc[b][s]));
          unpack8(to_uint4(regc[b][s]), x);
          if constexpr (MODE == 2) {
#pragma unroll
            for (int e = 0; e < 8; e++) x[e] = gc * x[e];
          }
          if constexpr (MOM) {
#pragma unroll
            for (int e = 0; e < 8; e++)
              x[e] = fmaf(k.a1, x[e], __fmul_rn(k.b1, __uint_as_float(momc[b][s][e / 4][e % 4])));
          }
#pragma unroll
          for (int e = 0; e < 8; e++) {
            const float ax = __fmul_rn(sc, x[e]);
            if (Z) {
              const double axd = (double)ax;
              zacc[s][e] = fma(axd * axd, winv, zacc[s][e]);
              amax = fmaxf(amax, fabsf(ax));
            }
            if (Y) {
              const float q0 = ax * reps;
              const float uf = fmaf(fmaf(-q0, deps, ax), reps, q0);   // RN(ax / deps)
              if (e & 1)
                ysum2 = fma((double)uf, (double)uf, ysum2);
              else
                ysum = fma((double)uf, (double)uf, ysum);
            }
          }
        }
        if (Z) umax = fmax(umax, ((double)amax * (double)amax) * winv);
        // a row with R_i == 0 but nonzero elements (mode 0 tests its sum instead)
        if (Z && MODE == 2 && winv == 0.0 && amax > 0.f) bad_l = 1;
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    // an idle wave (its rows are group 0's) adds nothing; mode 1 forms no update sums
    if constexpr (MODE != 1)
      if (active) sweep2(zc, yc);
  };
  u32x4_t regA[RB][NSEG], regB[RB][NSEG], momA[MB][MS][2], momB[MB][MS][2];
  float roldA = 0.f, roldB = 0.f;
  issue_g(0, regA, roldA);
  if constexpr (MDB) issue_m(0, momA);
  // the band's loop, specialised for the sums it forms (the regime is the same for the band)
  auto band_loop = [&](auto zc, auto yc) {
    for (int64_t blk = 0; blk < nblk; blk += 2) {
      step(blk, regA, roldA, momA, regB, roldB, momB, zc, yc);
      if (blk + 1 >= nblk) break;
      if constexpr (MDB)
        step(blk + 1, regB, roldB, momB, regA, roldA, momA, zc, yc);
      else
        step(blk + 1, regB, roldB, momA, regA, roldA, momA, zc, yc);
    }
  };
  if (MODE == 1 || (want_z && want_y))
    band_loop(std::true_type(), std::true_type());
  else if (want_z)
    band_loop(std::true_type(), std::false_type());
  else
    band_loop(std::false_type(), std::true_type());
  // column partials: the groups' sums added in group order through LDS, 16 chunks at a time,
  // then stored by consecutive threads
  auto store_cols = [&](const double (&acc)[NSEG][8], double *dst) {
    const int per = kColChunks / rpi;
    for (int c0 = 0; c0 < zcw; c0 += per) {
      const int nc = zcw - c0 < per ? zcw - c0 : per;
      __syncthreads();
      if (active) {
#pragma unroll
        for (int s = 0; s < NSEG; s++)
          if (chs[s] >= c0 && chs[s] < c0 + nc)
#pragma unroll
            for (int e = 0; e < 8; e++)
              colbuf[((grp * nc + chs[s] - c0) * 8 + e) * kColPad + lane] = acc[s][e];
      }
      __syncthreads();
      const int64_t cend = m - (int64_t)c0 * kChunk < (int64_t)nc * kChunk ? m - (int64_t)c0 * kChunk
                                                                          : (int64_t)nc * kChunk;
      for (int c = threadIdx.x; c < (int)cend; c += kZThreads) {
        const double *p = NARROW ? colbuf + c : colbuf + ((c >> 9) * 8 + (c & 7)) * kColPad + ((c >> 3) & 63);
        double v = p[0];
        for (int g = 1; g < rpi; g++) v += p[g * nc * 8 * kColPad];
        stg(dst + (int64_t)band * t.ldp + (int64_t)c0 * kChunk + c, v);
      }
    }
  };
  if constexpr (MODE != 2) store_cols(cacc, t.colpart);
  if constexpr (MODE != 1) store_cols(zacc, t.zpart);
  __syncthreads();   // every wave's rstash rows are there
  // the band's R and 1/sqrt(R) (coalesced), and its statistics: fixed-order reductions
  // (mode 1: the band's sum of g^2 instead; mode 2: R was written by the fold)
  double rs = rs_l;
  float rmn = __builtin_inff(), rmx = 0.f;
  if constexpr (MODE != 1)
    for (int j = threadIdx.x; j < (int)nblk * br; j += kZThreads) {
      const int64_t i = first_row(j / br) + j % br;
      if (i >= t.n) continue;
      const float R = rstash[j];
      const double Rd = (double)R;
      const bool normal = R > 0.f && R < __builtin_inff();
      if (MODE == 0) {
        stg(t.R + i, R);
        stg(t.ainv + i, normal ? rsq_d(Rd) : 1.0 / sqrt(Rd));
      }
      rs += Rd;
      if (R > 0.f) rmn = fminf(rmn, R);
      rmx = fmaxf(rmx, R);
    }
  // each wave reduces its values, thread 0 adds the waves in order (one barrier for all)
  const double ys = wave_sum_d(ysum + ysum2), um = wave_max_d(umax), rw = wave_sum_d(rs);
  const float rmin = wave_min_f(rmn), rmax = wave_max_f(rmx);
  const int bd = wave_or(bad_l);
  if (lane == 0) {
    double *o = sh + wave * kZStats;
    o[0] = ys;
    o[1] = um;
    o[2] = rw;
    o[3] = (double)rmin;
    o[4] = (double)rmax;
    o[5] = (double)bd;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a[kZStats];
    for (int q = 0; q < kZStats; q++) a[q] = sh[q];
    for (int w = 1; w < kZWaves; w++) {
      const double *o = sh + w * kZStats;
      a[0] += o[0];
      a[1] = fmax(a[1], o[1]);
      a[2] += o[2];
      a[3] = fmin(a[3], o[3]);
      a[4] = fmax(a[4], o[4]);
      a[5] = fmax(a[5], o[5]);
    }
    stg(&t.bst[band].ysum, a[0]);
    stg(&t.bst[band].umax, a[1]);
    stg(&t.bst[band].rsum, a[2]);
    stg(&t.bst[band].rmin, (float)a[3]);
    stg(&t.bst[band].rmax, (float)a[4]);
    stg(&t.bst[band].bad, (int32_t)(a[5] != 0.0));
    stg(&t.bst[band].regime, (int32_t)regime);
  }
}

// One launch covers the bands of every shape: a work-group fills a compute unit in all of
// them (two waves of up to 256 VGPRs per SIMD), so the bodies share a launch at no cost in
// occupancy, and the bands of a few small tensors run beside the others instead of after them.
template <int MODE>
__global__ __launch_bounds__(kZThreads) void p1z_kernel(const DevTensor *__restrict__ TT,
                                                        const Item *__restrict__ items, StepConsts k) {
  __shared__ double colbuf[kColChunks * 8 * kColPad];
  __shared__ double rowsh[2 * kZRowSlots];
  __shared__ double sh[kZWaves * kZStats];
  __shared__ float rstash[kZMaxBandRows + kZMaxBlockRows];
  const Item it = items[blockIdx.x];
  const DevTensor &t = TT[it.tensor];
  if (MODE != 1 && t.momentum) {
    constexpr bool M = MODE != 1;
    if (t.m < kZMinCols)
      p1z_body<1, zrows_per_group(1, true, MODE), M, MODE, true>(t, it.tile, k, colbuf, rowsh, sh, rstash);
    else if (t.nseg == 1)
      p1z_body<1, zrows_per_group(1, true, MODE), M, MODE>(t, it.tile, k, colbuf, rowsh, sh, rstash);
    else if (t.nseg == 2)
      p1z_body<2, zrows_per_group(2, true, MODE), M, MODE>(t, it.tile, k, colbuf, rowsh, sh, rstash);
    else
      p1z_body<4, zrows_per_group(4, true, MODE), M, MODE>(t, it.tile, k, colbuf, rowsh, sh, rstash);
  } else {   // (mode 1 reads no momentum: its rows per group do not depend on it)
    if (t.m < kZMinCols)
      p1z_body<1, zrows_per_group(1, false, MODE), false, MODE, true>(t, it.tile, k, colbuf, rowsh, sh, rstash);
    else if (t.nseg == 1)
      p1z_body<1, zrows_per_group(1, false, MODE), false, MODE>(t, it.tile, k, colbuf, rowsh, sh, rstash);
    else if (t.nseg == 2)
      p1z_body<2, zrows_per_group(2, false, MODE), false, MODE>(t, it.tile, k, colbuf, rowsh, sh, rstash);
    else if (t.nseg == 3)
      p1z_body<3, zrows_per_group(3, false, MODE), false, MODE>(t, it.tile, k, colbuf, rowsh, sh, rstash);
    else
      p1z_body<4, zrows_per_group(4, false, MODE), false, MODE>(t, it.tile, k, colbuf, rowsh, sh, rstash);
  }
}

// Reductions of the clip stage, over the whole work-group (a tensor of its own) or over one
// wave (the slices of a stacked tensor, one slice per wave at a time). Every participating
// lane gets the result, in a fixed order.
// What the clip stage reduces over a tensor or a slice: sums, a maximum, extremes and a flag. All of
// them in one exchange: one after the other, each with its barriers and its loads waited for on
// their own, they took the stage's 10 us (21 tensors) to 17 us (431).
struct RedAll {
  double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  double um = 0.0;
  float rmn = __builtin_inff(), cmn = __builtin_inff(), rmx = 0.f, cmx = 0.f;
  int bad = 0;
  __device__ __forceinline__ void wave() {
#pragma unroll
    for (int j = 0; j < 6; j++) s[j] = wave_sum_d(s[j]);
    um = wave_max_d(um);
    rmn = wave_min_f(rmn);
    cmn = wave_min_f(cmn);
    rmx = wave_max_f(rmx);
    cmx = wave_max_f(cmx);
    bad = wave_or(bad);
  }
};
struct RedGroup {
  double *sh;   // [kThreads]
  static constexpr int kN = kThreads;
  __device__ __forceinline__ int lane() const { return (int)threadIdx.x; }
  __device__ __forceinline__ bool lead() const { return threadIdx.x == 0; }
  __device__ __forceinline__ double sum(double x) const { return block_sum(x, sh); }
  __device__ __forceinline__ void all(RedAll &a) const {   // the waves in order
    constexpr int kVals = 12;
    static_assert(kVals * kWaves <= kThreads, "sh holds every wave's values");
    a.wave();
    if ((threadIdx.x & 63) == 0) {
      double *o = sh + (threadIdx.x >> 6) * kVals;
#pragma unroll
      for (int j = 0; j < 6; j++) o[j] = a.s[j];
      o[6] = a.um;
      o[7] = (double)a.rmn;
      o[8] = (double)a.cmn;
      o[9] = (double)a.rmx;
      o[10] = (double)a.cmx;
      o[11] = (double)a.bad;
    }
    __syncthreads();
    RedAll r;
#pragma unroll
    for (int w = 0; w < kWaves; w++) {
      const double *o = sh + w * kVals;
#pragma unroll
      for (int j = 0; j < 6; j++) r.s[j] += o[j];
      r.um = fmax(r.um, o[6]);
      r.rmn = fminf(r.rmn, (float)o[7]);
      r.cmn = fminf(r.cmn, (float)o[8]);
      r.rmx = fmaxf(r.rmx, (float)o[9]);
      r.cmx = fmaxf(r.cmx, (float)o[10]);
      r.bad |= o[11] != 0.0 ? 1 : 0;
    }
    __syncthreads();
    a = r;
  }
};
struct RedWave {
  static constexpr int kN = 64;
  __device__ __forceinline__ int lane() const { return (int)(threadIdx.x & 63); }
  __device__ __forceinline__ bool lead() const { return (threadIdx.x & 63) == 0; }
  __device__ __forceinline__ double sum(double x) const { return wave_sum_d(x); }
  __device__ __forceinline__ void all(RedAll &a) const { a.wave(); }
};
template <class Red>
__device__ __forceinline__ double red_sum(const Red &r, const double *p, int64_t n, int64_t stride = 1) {
  double s = 0.0;
  for (int64_t c = r.lane(); c < n; c += Red::kN) s += ldg(p + c * stride);
  return r.sum(s);
}

// fixed-order work-group sum of p[0], p[stride], ..., p[(n-1) stride]: thread j sums
// entries j, j + 256, ..., then a tree; every thread of the (256-thread) work-group calls it
__device__ __forceinline__ double wg_sum(const double *p, int64_t n, double *sh, int64_t stride = 1) {
  double s = 0.0;
  for (int64_t c = threadIdx.x; c < n; c += kThreads) s += ldg(p + c * stride);
  return block_sum(s, sh);
}
// q = max(mean R, eps) for a factored tensor (the clamp of the reconstruction), from the
// sums of R over the fold chunks of rows or over the row bands. Every kernel that forms it adds
// them in one order, that of a work-group of kThreads (lane j takes entries j, j + kThreads, ...;
// the lanes of a wave, then the waves in order): another one can round q to the other float, and
// c'_j = C_j / q would differ by 2^-24 between the sum that k comes from and the update.
__device__ __forceinline__ double sum_r_part(const DevTensor &t, const StepConsts &k, int lane) {
  // row-band tensors keep the sums of R in their band statistics, except in the gradient-
  // norm mode, where the fold forms R and its sums per chunk of rows as for wide tensors
  const bool bands = t.zpath && !k.gclip;
  const double *p = bands ? &t.bst->rsum : t.rsum;
  const int64_t n = bands ? t.nzb : (t.zpath ? (t.n + kFold - 1) / kFold : t.nfr);
  const int64_t stride = bands ? sizeof(BandStats) / sizeof(double) : 1;
  double s = 0.0;   // the lane's share
  for (int64_t c = lane; c < n; c += kThreads) s += ldg(p + c * stride);
  return s;
}
__device__ __forceinline__ double sum_r_wave(const DevTensor &t, const StepConsts &k) {   // by one wave
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < kWaves; w++) s += wave_sum_d(sum_r_part(t, k, w * 64 + (int)(threadIdx.x & 63)));
  return s;
}
__device__ __forceinline__ float mean_r_from(const DevTensor &t, const StepConsts &k, double sr) {
  return max_nan((float)(sr / (double)t.n), k.eps);
}
__device__ __forceinline__ float mean_r_clamped(const DevTensor &t, const StepConsts &k, double *sh) {
  return mean_r_from(t, k, block_sum(sum_r_part(t, k, (int)threadIdx.x), sh));
}

// --------------------------------------------------------------------------------------------
// fold: R_i <- b2 R_i + a2 r_i, C_j <- b2 C_j + a2 c_j (Eq. 1), 1/sqrt(R_i), sums of R
//
// A chain of dependent loads bounds it, not their bytes: a thread that adds the partials of
// every band by itself waits for them a few at a time (786 bands of a 50304-row embedding). So
// kFoldParts groups of threads each add a quarter of the partials (bands or strips) of a
// chunk of kFold rows or columns, two per thread, and the quarters are added in order through
// LDS. Each wave reduces its statistics and thread 0 adds the waves' in order: one barrier for
// all of them.
// --------------------------------------------------------------------------------------------
constexpr int kFoldParts = 4;
constexpr int kFoldThreads = kFold / 2 * kFoldParts;

struct FoldShared {
  double part[2][kFoldParts][kFold];
  double stat[kFoldThreads / 64][8];
  float nb[kFold];
  double rsum[kWaves];
  int dup[kFoldThreads / 64];
};
// The sums of a[p * stride + x0 + c] over p = 0 .. n - 1 (and of b) for the columns x0 + c < xn of
// a chunk: two columns per thread (16-byte loads), the p split in kFoldParts runs of their own,
// added in order through LDS. Thread c < kFold gets its column's totals. Every thread calls it.
typedef double f64x2_t __attribute__((ext_vector_type(2), aligned(8)));
template <bool TWO>
__device__ __forceinline__ void fold_sum(const double *a, const double *b, int n, int64_t stride, int64_t x0,
                                         int64_t xn, FoldShared &f, double &as, double &bs) {
  constexpr int half = kFold / 2, U = 4;
  const int c = (threadIdx.x & (half - 1)) * 2, part = threadIdx.x / half;
  const int per = (n + kFoldParts - 1) / kFoldParts, p0 = part * per, p1 = p0 + per < n ? p0 + per : n;
  f64x2_t x = {0.0, 0.0}, y = {0.0, 0.0};
  if (x0 + c < xn) {
    // (the last column of an odd row is loaded with the one before it)
    const int64_t at0 = x0 + c + 1 < xn || x0 + c == 0 ? x0 + c : x0 + c - 1;
    const bool back = at0 != x0 + c;
    const bool one = xn == 1;
    auto load = [&](const double *p) {
      f64x2_t v = {0.0, 0.0};
      if (one)
        v.x = ldg(p);
      else
        v = *(const __attribute__((address_space(1))) f64x2_t *)p;
      if (back) v.x = v.y;
      return v;
    };
    // loads of several bands in flight (past the last, of the last again: not added); the sums
    // run in band order
    for (int p = p0; p < p1; p += U) {
      f64x2_t va[U], vb[U];
#pragma unroll
      for (int u = 0; u < U; u++) {
        const int64_t at = (int64_t)(p + u < p1 ? p + u : p1 - 1) * stride + at0;
        va[u] = load(a + at);
        if constexpr (TWO) vb[u] = load(b + at);
      }
#pragma unroll
      for (int u = 0; u < U; u++)
        if (p + u < p1) {
          x += va[u];
          if constexpr (TWO) y += vb[u];
        }
    }
  }
  f.part[0][part][c] = x.x;
  f.part[0][part][c + 1] = x.y;
  if constexpr (TWO) {
    f.part[1][part][c] = y.x;
    f.part[1][part][c + 1] = y.y;
  }
  __syncthreads();
  as = bs = 0.0;
  if (threadIdx.x < kFold)
#pragma unroll
    for (int q = 0; q < kFoldParts; q++) {
      as += f.part[0][q][threadIdx.x];
      if constexpr (TWO) bs += f.part[1][q][threadIdx.x];
    }
}
// Extremes of the positive values and equal neighbours within one fold chunk (v of this
// thread's row or column, 0 past the end), for the clip stage's test of repeated factors, and
// the sum of s; every thread calls it, those of part 0 with their values
__device__ __forceinline__ void chunk_stats(ColStats *out, double *sum_out, float v, double s, FoldShared &f) {
  const int c = threadIdx.x & (kFold - 1);
  const bool own = threadIdx.x < kFold;
  if (own) f.nb[c] = v;
  __syncthreads();
  if (own) {
    const double dup = wave_sum_d((c > 0 && v > 0.f && v == f.nb[c - 1]) ? 1.0 : 0.0), tot = wave_sum_d(s);
    const float mn = wave_min_f(v > 0.f ? v : __builtin_inff()), mx = wave_max_f(v);
    if ((threadIdx.x & 63) == 0) {
      double *o = f.stat[threadIdx.x >> 6];
      o[0] = dup;
      o[1] = tot;
      o[2] = (double)mn;
      o[3] = (double)mx;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double d = 0.0, tot = 0.0, mn = __builtin_inf(), mx = 0.0;
    for (int w = 0; w < kFold / 64; w++) {
      d += f.stat[w][0];
      tot += f.stat[w][1];
      mn = fmin(mn, f.stat[w][2]);
      mx = fmax(mx, f.stat[w][3]);
    }
    if (out != nullptr) {
      stg(&out->cmin, (float)mn);
      stg(&out->cmax, (float)mx);
      stg(&out->cdup, (int32_t)d);
    }
    if (sum_out != nullptr) stg(sum_out, tot);
  }
}

// Repeated row factors of a row-band tensor: in rows [chunk kZMaxBandRows, ...), those whose R_i > 0
// equals R_{i-1}. (A band's blocks of rows lie apart, so the row-band pass cannot tell: its blocks
// are single rows where a row takes the whole work-group.) A tensor of one such run has it counted
// by its first column chunk: work-groups of their own took the fold of 512 slices of 16 x 512 from
// 6.9 to 10.2 us (8.5 so). Its loads follow the partials': ahead of them they cost the fold of the
// 6.78B set 4 us more (79 instead of 75; 71 without the count), for the registers that they hold.
struct EqualRows {
  static constexpr int kPer = kZMaxBandRows / kFoldThreads;
  float a[kPer], b[kPer];
  __device__ __forceinline__ void load(const DevTensor &t, int chunk) {
#pragma unroll
    for (int q = 0; q < kPer; q++) {
      const int64_t i0 = (int64_t)chunk * kZMaxBandRows + q * kFoldThreads, i = i0 + threadIdx.x;
      a[q] = b[q] = 0.f;
      if (i0 < t.n) {   // (uniform)
        const bool in = i > 0 && i < t.n;
        a[q] = ldg(t.R + (in ? i : 0));
        b[q] = in ? ldg(t.R + (in ? i - 1 : 0)) : -1.f;
      }
    }
  }
  // each wave's share goes to f.dup; a barrier later thread 0 stores their sum
  __device__ __forceinline__ void count(FoldShared &f) const {
    int n = 0;   // of the wave (uniform)
#pragma unroll
    for (int q = 0; q < kPer; q++) n += __popcll(__ballot(a[q] > 0.f && a[q] == b[q]));
    if ((threadIdx.x & 63) == 0) f.dup[threadIdx.x >> 6] = n;
  }
  static __device__ __forceinline__ void store(const DevTensor &t, int chunk, const FoldShared &f) {
    int all = 0;
    for (int w = 0; w < kFoldThreads / 64; w++) all += f.dup[w];
    stg(&t.bst[chunk].rdup, (int32_t)all);
  }
};

__global__ __launch_bounds__(kFoldThreads) __attribute__((amdgpu_waves_per_eu(8))) void fold_kernel(const DevTensor *__restrict__ TT,
                                                            const Item *__restrict__ items, StepConsts k, int phase) {
  __shared__ FoldShared f;
  const Item it = items[blockIdx.x];
  const DevTensor &t = TT[it.tensor];
  // gradient-norm mode: the statistics of the scaled gradient are c^2 times the exact sums
  const double c2 = phase == 1 ? (double)ldg(k.gscale) * (double)ldg(k.gscale) : 1.0;
  // row chunks of this launch: wide tensors always; row-band tensors only in phase 1,
  // where their row sums of g^2 wait in ainv
  const int nrows = t.zpath ? (phase == 1 ? (int)((t.n + kFold - 1) / kFold) : 0) : t.nfr;
  if (phase == 2 && !t.zpath) return;
  if (t.zpath && phase != 1 && it.tile >= t.nfc) {   // (R is final: from the row-band pass or from phase 1)
    EqualRows eq;
    eq.load(t, it.tile - t.nfc);
    eq.count(f);
    __syncthreads();
    if (threadIdx.x == 0) EqualRows::store(t, it.tile - t.nfc, f);
    return;
  }
  const int c = threadIdx.x & (kFold - 1);   // the row or column of the chunk that an `own` thread ends with
  const bool own = threadIdx.x < kFold;
  if (it.tile < nrows) {
    const int64_t i = (int64_t)it.tile * kFold + c;
    double s, none, rn = 0.0;
    fold_sum<false>(t.zpath ? t.ainv : t.rowpart, nullptr, t.zpath ? 1 : t.ntc, t.n, i - c, t.n, f, s, none);
    float Rv = 0.f;
    if (own && i < t.n) {
      const float ri = (float)((phase == 1 ? c2 * s : s) / (double)t.m);
      const float R = fmaf(k.a2, ri, __fmul_rn(k.b2, ldg(t.R + i)));
      stg(t.R + i, R);
      stg(t.ainv + i, 1.0 / sqrt((double)R));
      rn = (double)R;
      Rv = R;
    }
    chunk_stats(t.zpath ? nullptr : t.cst + it.tile, t.rsum + it.tile, Rv, rn, f);
  } else if (!t.zpath || phase == 1) {
    // C_j from the column partials ([row bands][m] of either pass 1)
    const int64_t j = (int64_t)(it.tile - nrows) * kFold + c;
    double s, none;
    fold_sum<false>(t.colpart, nullptr, t.zpath ? t.nzb : t.ntr, t.ldp, j - c, t.m, f, s, none);
    float Cv = 0.f;
    if (own && j < t.m) {
      const float cj = (float)((phase == 1 ? c2 * s : s) / (double)t.n);
      Cv = fmaf(k.a2, cj, __fmul_rn(k.b2, ldg(t.C + j)));
      stg(t.C + j, Cv);
    }
    if (!t.zpath) chunk_stats(t.cst + t.nfr + (it.tile - nrows), nullptr, Cv, 0.0, f);
  } else {
    // row-band tensor: C_j (phase 0; phase 2 has it from phase 1), c'_j = C_j / max(mean R,
    // eps) and sum_j z_j / c'_j over the chunk; the first waves add the sums of R while the
    // partials load (fold_sum's barrier covers theirs)
    const bool count = it.tile == 0 && t.n <= kZMaxBandRows;
    if (threadIdx.x < kThreads) {
      const double sr = wave_sum_d(sum_r_part(t, k, (int)threadIdx.x));
      if ((threadIdx.x & 63) == 0) f.rsum[threadIdx.x >> 6] = sr;
    }
    const int64_t j = (int64_t)it.tile * kFold + c;
    double cs, zs;
    fold_sum<true>(t.colpart, t.zpart, t.nzb, t.ldp, j - c, t.m, f, cs, zs);
    EqualRows eq;
    if (count) eq.load(t, 0);
    double sr = 0.0;
    for (int w = 0; w < kWaves; w++) sr += f.rsum[w];
    const float q = mean_r_from(t, k, sr);
    if (it.tile == 0 && threadIdx.x == 0) stg(&t.sc->q, q);   // for the clip stage and the update
    double sj = 0.0, sj2 = 0.0;
    float cmn = __builtin_inff(), cmx = 0.f, Cj = 0.f;
    int bad = 0;
    if (own && j < t.m) {
      float C;
      if (phase == 0) {
        const float cj = (float)(cs / (double)t.n);
        C = fmaf(k.a2, cj, __fmul_rn(k.b2, ldg(t.C + j)));
        stg(t.C + j, C);
      } else {
        C = ldg(t.C + j);
      }
      Cj = C;
      const float cp = C / q;
      if (C > 0.f) {
        // c'_j that is zero or not finite leaves the tensor to the exact pass
        if (cp > 0.f && cp < __builtin_inff()) {
          sj = zs / (double)cp;
          sj2 = sj / (double)cp;
          cmn = cmx = cp;
        } else {
          bad = 1;
        }
      } else if (C != 0.f || cs > 0.0 || zs > 0.0) {
        bad = 1;   // NaN, or a nonzero column whose C underflowed
      }
    }
    if (count) eq.count(f);
    // repeated column factors: C_j equal to the previous column's (within the chunk)
    if (own) f.nb[c] = Cj;
    __syncthreads();
    if (own) {
      const double S = wave_sum_d(sj), S2 = wave_sum_d(sj2);
      const double dup = wave_sum_d((c > 0 && Cj > 0.f && Cj == f.nb[c - 1]) ? 1.0 : 0.0);
      const float mn = wave_min_f(cmn), mx = wave_max_f(cmx);
      const int b = wave_or(bad);
      if ((threadIdx.x & 63) == 0) {
        double *o = f.stat[threadIdx.x >> 6];
        o[0] = S;
        o[1] = S2;
        o[2] = dup;
        o[3] = (double)mn;
        o[4] = (double)mx;
        o[5] = (double)b;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      double S = 0.0, S2 = 0.0, dup = 0.0, mn = __builtin_inf(), mx = 0.0, b = 0.0;
      for (int w = 0; w < kFold / 64; w++) {
        const double *o = f.stat[w];
        S += o[0];
        S2 += o[1];
        dup += o[2];
        mn = fmin(mn, o[3]);
        mx = fmax(mx, o[4]);
        b = fmax(b, o[5]);
      }
      ColStats *o = t.cst + it.tile;
      stg(&o->cdup, (int32_t)dup);
      stg(&o->s2, S2);
      stg(&o->s, S);
      stg(&o->cmin, (float)mn);
      stg(&o->cmax, (float)mx);
      stg(&o->bad, (int32_t)(b != 0.0));
      if (count) EqualRows::store(t, 0, f);
    }
  }
}

// Gradient-norm mode: sum of g^2 of each (tile, part) of an exact tensor, into its update-sum
// slot (the update-sum pass later overwrites it); factored items have theirs in pass 1
__global__ __launch_bounds__(kThreads) void gsq_kernel(const DevTensor *__restrict__ TT,
                                                       const Item *__restrict__ items) {
  __shared__ double sh[kThreads];
  const Item it = items[blockIdx.x];   // it.tile = tile * kSub + part
  const DevTensor &t = TT[it.tensor];
  if (t.kind == kFactored) return;
  const Tile tl = tile_of(t, it.tile / kSub);
  const WaveMap wm(t, tl);
  const int64_t r0 = wm.wr + (int64_t)(it.tile % kSub) * wm.rpi, rs = (int64_t)wm.rpi * kSub;
  const Cols8 cols(t.m, wm.col);
  double acc = 0.0;
  for (int64_t lr = r0; wm.col < t.m && lr < tl.nr; lr += rs) {
    const int64_t i = tl.row(lr);
    float g[8];
    load_elems8(t.g, i * t.ld, cols, t.fp32, g);
#pragma unroll
    for (int e = 0; e < 8; e++) acc += (double)g[e] * (double)g[e];   // (0 past the row's end)
  }
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0) stg(t.ssum + it.tile, s);
}

// Gradient-norm mode: ||G||^2 of each tensor (one work-group per tensor), then over the
// table in table order and the scale c = min(1, max_grad_norm / (||G|| + 1e-6)) (NaN
// propagates; one work-group)
__global__ __launch_bounds__(kThreads) void gsum_kernel(const DevTensor *__restrict__ TT, StepConsts k) {
  __shared__ double sh[kThreads];
  const DevTensor &t = TT[blockIdx.x];
  double s = 0.0;
  if (t.n * t.m > 0) {
    if (t.kind != kFactored)
      s = wg_sum(t.ssum, (int64_t)t.ntr * t.ntc * kSub, sh);
    else if (t.zpath)
      s = wg_sum(&t.bst->rsum, t.nzb, sh, sizeof(BandStats) / sizeof(double));
    else
      s = wg_sum(t.rowpart, (int64_t)t.ntc * t.n, sh);
  }
  if (threadIdx.x == 0) stg(k.gsq + blockIdx.x, s);
}
__global__ __launch_bounds__(kThreads) void gnorm_kernel(int ntensors, StepConsts k) {
  __shared__ double sh[kThreads];
  const double total = wg_sum(k.gsq, ntensors, sh);
  if (threadIdx.x == 0) {
    double c = (double)k.max_grad_norm / (sqrt(total) + 1e-6);
    if (c > 1.0) c = 1.0;
    stg(k.gscale, (float)c);
  }
}

// Column factors of the rank-one reconstruction: q = max(mean R, eps) and c'_j = C_j / q
// rounded as the oracle rounds them; b_j = 1/sqrt(c'_j) in double, so that
// 1/D_ij = min(b_j / sqrt(R_i), 1/sqrt(eps)) (Eq. 1 reconstruction with the Alg. 1 clamps).
__device__ __forceinline__ double col_factor(const DevTensor &t, int64_t col, float q) {
  return 1.0 / sqrt((double)(ldg(t.C + col) / q));
}

// --------------------------------------------------------------------------------------------
// p2: per-tile sum of squares of the unclipped update U_hat (Alg. 1, before clipping).
//
// The clip factor must round to the oracle's float, so the sum must match the oracle's
// sum of its rounded U_hat to ~1e-13. Roundings that repeat a pattern are replicated
// exactly: s*x (a fixed s times 8-bit bf16 mantissas) and, on the floor, the division
// by the constant D = sqrt(eps) (Markstein's correctly rounded division with the
// correctly rounded reciprocal). Above the floor the oracle's three roundings (of R_i c'_j,
// the square root and the quotient) vary freely from element to element, so U_hat is
// taken unrounded in double, and the sum of U_hat^4 over those elements gives the
// spread of the difference. The clip stage decides k from this; when the bound leaves
// k's rounding open, an exact pass (p2_exact) recomputes the tensor's sum.
// --------------------------------------------------------------------------------------------
struct SumPair {
  double s, q4;
};

template <bool NT = false>
__device__ __forceinline__ SumPair p2_factored(const DevTensor &t, const Tile &tl, int part, const StepConsts &k,
                                               float q) {
  const WaveMap wm(t, tl);
  const int64_t r0 = wm.wr + (int64_t)part * wm.rpi, rs = (int64_t)wm.rpi * kSub;   // this part's rows
  const int64_t m = t.m, ld = t.ld, col = wm.col;
  const bool mom = t.momentum != 0;
  const float s = mom ? k.s_m : k.s_0;
  const float deps = sqrtf(k.eps);                    // the oracle's D on the floor
  const float reps = (float)(1.0 / (double)deps);     // correctly rounded 1/D
  const float gc = k.gclip ? ldg(k.gscale) : 1.f;     // gradient-norm mode: elements are fl(c g)
  SumPair acc = {0.0, 0.0};
  if (col >= m) return acc;
  const Cols8 cols(m, col);
  float cp[8];    // c'_j = C_j / q, rounded as the oracle (1 past the row's end, where x is 0)
  double bd[8];   // 1/sqrt(c'_j) to about 2^-50 (it scales the unrounded estimate only)
#pragma unroll
  for (int e = 0; e < 8; e++) {
    cp[e] = (col + e < m) ? ldg(t.C + col + e) / q : 1.f;
    const double cd = (double)cp[e];
    bd[e] = (cp[e] > 0.f && cp[e] < __builtin_inff()) ? rsq_d(cd) : 1.0 / sqrt(cd);
  }
  auto elem = [&](float x, float Ri, double ai, int e, SumPair &a) {
    const float ax = __fmul_rn(s, x);
    const bool floored = __fmul_rn(Ri, cp[e]) < k.eps;
    const float q0 = ax * reps;
    const float uf = fmaf(fmaf(-q0, deps, ax), reps, q0);   // RN(ax / deps)
    const double ud = (double)ax * (ai * bd[e]);
    const double u = floored ? (double)uf : ud;
    a.s = fma(u, u, a.s);
    const double u2 = floored ? 0.0 : ud * ud;
    a.q4 = fma(u2, u2, a.q4);
  };
  for (int64_t lr = r0; lr < tl.nr; lr += 2 * rs) {
    const bool two = lr + rs < tl.nr;
    const int64_t i = tl.row(lr), i2 = two ? tl.row(lr + rs) : i;
    const u32x4_t ga = load8<NT>(t.g + i * ld, cols), gb = load8<NT>(t.g + i2 * ld, cols);
    float ma[8], mb[8];
    if (mom) {
      load8(t.M + i * m, cols, ma);
      load8(t.M + i2 * m, cols, mb);
    }
    const float Ra = ldg(t.R + i), Rb = ldg(t.R + i2);
    const double aa = ldg(t.ainv + i), ab = ldg(t.ainv + i2);
    float xa[8], xb[8];
    unpack8(to_uint4(ga), xa);
    unpack8(to_uint4(gb), xb);
    if (k.gclip) {
#pragma unroll
      for (int e = 0; e < 8; e++) {
        xa[e] = gc * xa[e];
        xb[e] = gc * xb[e];
      }
    }
    if (mom) {
#pragma unroll
      for (int e = 0; e < 8; e++) {
        xa[e] = fmaf(k.a1, xa[e], __fmul_rn(k.b1, ma[e]));
        xb[e] = fmaf(k.a1, xb[e], __fmul_rn(k.b1, mb[e]));
      }
    }
    SumPair sa = {0.0, 0.0}, sb = {0.0, 0.0};
#pragma unroll
    for (int e = 0; e < 8; e++) {
      elem(xa[e], Ra, aa, e, sa);
      elem(xb[e], Rb, ab, e, sb);
    }
    acc.s += sa.s;
    acc.q4 += sa.q4;
    if (two) {
      acc.s += sb.s;
      acc.q4 += sb.q4;
    }
  }
  return acc;
}

// The oracle's own float sequence for U_hat of a factored tensor, summed in double:
// used when the approximate sum leaves the clip factor's rounding undecided.
__device__ __forceinline__ double p2_factored_exact(const DevTensor &t, const Tile &tl, int part,
                                                    const StepConsts &k, float q) {
  const WaveMap wm(t, tl);
  const int64_t r0 = wm.wr + (int64_t)part * wm.rpi, rs = (int64_t)wm.rpi * kSub;
  const int64_t m = t.m, ld = t.ld, col = wm.col;
  const bool mom = t.momentum != 0;
  const float s = mom ? k.s_m : k.s_0;
  const float gc = k.gclip ? ldg(k.gscale) : 1.f;
  double acc = 0.0;
  if (col >= m) return 0.0;
  const Cols8 cols(m, col);
  float cp[8];   // (1 past the row's end, where x is 0)
#pragma unroll
  for (int e = 0; e < 8; e++) cp[e] = (col + e < m) ? ldg(t.C + col + e) / q : 1.f;
  for (int64_t lr = r0; lr < tl.nr; lr += rs) {
    const int64_t i = tl.row(lr);
    const float Ri = ldg(t.R + i);
    float x[8], mo[8];
    unpack8(to_uint4(load8(t.g + i * ld, cols)), x);
    if (mom) load8(t.M + i * m, cols, mo);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      // the momentum update takes the scaled gradient (as in the update pass)
      const float xs = k.gclip ? gc * x[e] : x[e];
      const float xm = mom ? fmaf(k.a1, xs, __fmul_rn(k.b1, mo[e])) : xs;
      const float u = __fmul_rn(s, xm) / sqrtf(max_nan(__fmul_rn(Ri, cp[e]), k.eps));
      acc = fma((double)u, (double)u, acc);
    }
  }
  return acc;
}

__device__ __forceinline__ double p2_exact(const DevTensor &t, const Tile &tl, int part, const StepConsts &k) {
  // exact second moment (router tier, vectors): the oracle's operation order exactly
  const WaveMap wm(t, tl);
  const int64_t r0 = wm.wr + (int64_t)part * wm.rpi, rs = (int64_t)wm.rpi * kSub;
  const int64_t m = t.m, ld = t.ld, col = wm.col;
  const bool mom = t.momentum != 0;
  const float gc = k.gclip ? ldg(k.gscale) : 1.f;
  const Cols8 cols(m, col);
  double acc = 0.0;
  for (int64_t lr = r0; col < m && lr < tl.nr; lr += rs) {
    const int64_t i = tl.row(lr);
    float g[8], v[8], mo[8];
    load_elems8(t.g, i * ld, cols, t.fp32, g);
    load8(t.V + i * m, cols, v);
    if (mom) load8(t.M + i * m, cols, mo);
#pragma unroll
    for (int e = 0; e < 8; e++) {   // (0 past the row's end)
      if (k.gclip) g[e] = gc * g[e];
      const float vn = fmaf(k.a2, __fmul_rn(g[e], g[e]), __fmul_rn(k.b2, v[e]));
      const float dd = sqrtf(max_nan(vn, k.eps));
      const float num = mom ? __fmul_rn(k.s_m, fmaf(k.a1, g[e], __fmul_rn(k.b1, mo[e]))) : __fmul_rn(k.s_0, g[e]);
      const float u = num / dd;
      acc += (double)u * (double)u;
    }
  }
  return acc;
}

__global__ __launch_bounds__(kThreads) void p2_kernel(const DevTensor *__restrict__ TT,
                                                      const Item *__restrict__ items, StepConsts k) {
  __shared__ double sh[kThreads];
  const Item it = items[blockIdx.x];   // it.tile = tile * kSub + part
  const DevTensor &t = TT[it.tensor];
  const Tile tl = tile_of(t, it.tile / kSub);
  const int part = it.tile % kSub;
  SumPair acc;
  if (t.kind == kFactored) {
    const float q = mean_r_clamped(t, k, sh);
    // (with momentum the rows of M push G out of the caches anyway, and the hint keeps some of M there:
    // 2048 x 50304 in a table of 1.6e9 elements 125 us without it, 122 with; step of 3355 x 20000 331, 324)
    acc = t.momentum ? p2_factored<true>(t, tl, part, k, q) : p2_factored<false>(t, tl, part, k, q);
  } else {
    acc.s = p2_exact(t, tl, part, k);   // already the oracle's own U_hat
    acc.q4 = 0.0;
  }
  const double s = block_sum(acc.s, sh);
  const double q4 = block_sum(acc.q4, sh);
  if (threadIdx.x == 0) {
    stg(t.ssum + it.tile, s);
    stg(t.qsum + it.tile, q4);
  }
}

// Re-check of the listed tensors over their tiles: level 1 forms the update sum with the
// exact floor test per element (the floored part exactly rounded, the rest unrounded, and
// the sum of U_hat^4 over the rest for its spread); level 2 follows the oracle's float
// sequence exactly. A fixed grid walks the (tensor, tile) pairs of the list.
__device__ __forceinline__ int32_t *recheck_list(RecheckLists *L, int ntensors, int level) {
  int32_t *l1 = reinterpret_cast<int32_t *>(L + 1);
  return level == 1 ? l1 : l1 + ntensors;
}

__global__ __launch_bounds__(kThreads) void recheck_kernel(const DevTensor *__restrict__ TT, RecheckLists *L,
                                                           int ntensors, StepConsts k, int level) {
  __shared__ double sh[kThreads];
  // tile offsets of the listed tensors (an exclusive prefix sum), when the list fits
  constexpr int kTable = 2048;
  __shared__ int64_t pre[kTable + 1];
  __shared__ int64_t part[kThreads];
  const int n = ldg(level == 1 ? &L->n1 : &L->n2);
  if (n <= 0) return;
  const int32_t *list = recheck_list(L, ntensors, level);
  auto tiles = [&](int j) {
    const int32_t ti = ldg(list + j);
    if (ti < 0) return (int64_t)0;   // a slice of a stack whose fast sum is kept
    const DevTensor &t = TT[ti];
    return (int64_t)t.ntr * t.ntc * kSub;   // per-part sums
  };
  const bool table = n <= kTable;
  int64_t total = 0;
  if (table) {
    // thread i sums the counts of entries [8i, 8i + 8), a scan over the threads gives each
    // its start, and it writes its entries' offsets
    constexpr int kPer = kTable / kThreads;
    const int j0 = (int)threadIdx.x * kPer;
    int64_t c[kPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kPer; q++) {
      c[q] = j0 + q < n ? tiles(j0 + q) : 0;
      sum += c[q];
    }
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < kThreads; off <<= 1) {   // inclusive scan of the thread sums
      const int64_t v = threadIdx.x >= (unsigned)off ? part[threadIdx.x - off] : 0;
      __syncthreads();
      part[threadIdx.x] += v;
      __syncthreads();
    }
    int64_t run = part[threadIdx.x] - sum;
#pragma unroll
    for (int q = 0; q < kPer; q++) {
      pre[j0 + q] = run;
      run += c[q];
    }
    if (threadIdx.x == kThreads - 1) pre[kTable] = run;
    __syncthreads();
    total = pre[n];
  } else {
    for (int j = 0; j < n; j++) total += tiles(j);
  }
  // the tiles of this work-group come in increasing order, so the listed tensor they fall
  // in only moves forward; q is formed once per tensor
  int j = 0, qj = -1;
  int64_t base = 0, nt_j = table ? pre[1] - pre[0] : tiles(0);
  float q = 0.f;
  for (int64_t idx = blockIdx.x; idx < total; idx += gridDim.x) {
    while (idx >= base + nt_j) {
      base += nt_j;
      j++;
      nt_j = table ? pre[j + 1] - pre[j] : tiles(j);
    }
    const DevTensor &t = TT[ldg(list + j)];
    const int tile = (int)(idx - base);   // tile * kSub + part
    const Tile tl = tile_of(t, tile / kSub);
    const int prt = tile % kSub;
    if (j != qj) {
      q = ldg(&t.sc->q);   // the clip stage's q (the one the update pass takes)
      qj = j;
    }
    if (level == 1) {
      const SumPair acc = p2_factored(t, tl, prt, k, q);
      const double sv = block_sum(acc.s, sh);
      const double q4 = block_sum(acc.q4, sh);
      if (threadIdx.x == 0) {
        stg(t.ssum + tile, sv);
        stg(t.qsum + tile, q4);
      }
    } else {
      const double sv = block_sum(p2_factored_exact(t, tl, prt, k, q), sh);
      if (threadIdx.x == 0) stg(t.ssum + tile, sv);
    }
  }
}

// k = 1 / max(1, RMS / d) from the sum S over N elements, rounded once to float (NaN
// propagates); `amb` when a relative spread of S may move k across a rounding boundary of
// the float or across the clipping threshold
__device__ __forceinline__ float clip_from_sum(double S, double N, float d, double spread, bool &amb) {
  const double r = sqrt(S / N) / (double)d;
  const double den = (r != r) ? r : (r < 1.0 ? 1.0 : r);
  const double kd = 1.0 / den;
  const float kf = (float)kd;
  if (!amb && S > 0.0 && r == r && r < 1e300 && spread > 0.0) {
    if (fabs(r - 1.0) <= spread) amb = true;   // at the clipping threshold
    if (r > 1.0) {
      const double up = (double)nextafterf(kf, 3.0e38f), dn = (double)nextafterf(kf, 0.f);
      const double mid_hi = 0.5 * ((double)kf + up), mid_lo = 0.5 * ((double)kf + dn);
      const double tol = 0.5 * spread * kd;
      if (fabs(kd - mid_hi) <= tol || fabs(kd - mid_lo) <= tol) amb = true;
    }
  }
  return kf;
}

// clip factors of the listed tensors from the re-check's sums; level 1 lists for level 2
// the tensors whose spread still leaves k undecided. A stacked tensor's slices are listed
// together; the work-group of its first slice decides k for all of them (one slice per
// wave at a time), the others return.
__global__ __launch_bounds__(kThreads) void clip_recheck_kernel(const DevTensor *__restrict__ TT, RecheckLists *L,
                                                                int ntensors, StepConsts k, int level) {
  __shared__ double sh[kThreads];
  __shared__ double wsum[kWaves][3];
  __shared__ double wek[kWaves];
  __shared__ float kf_sh;
  __shared__ int amb_sh, pos_sh;
  const int n = ldg(level == 1 ? &L->n1 : &L->n2);
  if ((int)blockIdx.x >= n) return;
  const int ti = ldg(recheck_list(L, ntensors, level) + blockIdx.x);
  if (ti < 0) return;
  const DevTensor &t0 = TT[ti];
  if (t0.grp0 != ti) return;
  const int ng = t0.ngrp;
  double S = 0.0, Q4 = 0.0, N = 0.0, Ek = 0.0;   // Ek: error bounds of the kept fast sums
  if (ng == 1) {
    const int64_t ntiles = (int64_t)t0.ntr * t0.ntc * kSub;   // per-part sums
    S = red_sum(RedGroup{sh}, t0.ssum, ntiles);
    if (level == 1) Q4 = red_sum(RedGroup{sh}, t0.qsum, ntiles);
    N = (double)(t0.n * t0.m);
  } else {
    // level 1 re-read only the stack's open slices (and its first); the others, listed as
    // -1 (the group's entries are consecutive from this one), keep the clip stage's fast
    // sum and its error bound
    const int w = (int)(threadIdx.x >> 6);
    double s = 0.0, q4 = 0.0, nn = 0.0, ek = 0.0;
    for (int e = w; e < ng; e += kWaves) {
      const DevTensor &t = TT[ti + e];
      const int64_t ntiles = (int64_t)t.ntr * t.ntc * kSub;
      if (level == 1 && ldg(recheck_list(L, ntensors, 1) + blockIdx.x + e) < 0) {
        s += ldg(&t.sc->s_fast);
        ek += ldg(&t.sc->e_fast);
      } else {
        s += red_sum(RedWave{}, t.ssum, ntiles);
        if (level == 1) q4 += red_sum(RedWave{}, t.qsum, ntiles);
      }
      nn += (double)(t.n * t.m);
    }
    if ((threadIdx.x & 63) == 0) {
      wsum[w][0] = s;
      wsum[w][1] = q4;
      wsum[w][2] = nn;
      wek[w] = ek;
    }
    __syncthreads();
    for (int v = 0; v < kWaves; v++) {   // waves in order
      S += wsum[v][0];
      Q4 += wsum[v][1];
      N += wsum[v][2];
      Ek += wek[v];
    }
  }
  if (threadIdx.x == 0) {
    bool amb = false;
    const double spread = level == 1 ? (20.0 * 0x1p-23 * sqrt(Q4) + Ek) / S + 1e-14 : 0.0;
    if (level == 1) stg(&t0.sc->split_spread, (float)spread);   // for the next step's routing
    kf_sh = clip_from_sum(S, N, k.d, spread, amb);
    amb_sh = amb;
    pos_sh = amb ? atomicAdd(&L->n2, ng) : 0;
  }
  __syncthreads();
  const float kf = kf_sh;
  const bool amb = amb_sh != 0;
  const int pos = pos_sh;
  const int why = ldg(&t0.sc->ambiguous) & ~0xF;
  for (int e = (int)threadIdx.x; e < ng; e += kThreads) {
    if (amb) {
      stg(recheck_list(L, ntensors, 2) + pos + e, (int32_t)(ti + e));
      stg(&TT[ti + e].sc->ambiguous, (int32_t)(kClipPending2 | (kWhySpread << 4)));
    } else {
      stg(&TT[ti + e].sc->k, kf);
      stg(&TT[ti + e].sc->ambiguous, (int32_t)(why | (level == 1 ? kClipSplit : kClipExact)));
    }
  }
}

// One slice's share of the clip stage (a tensor, or one slice of a stacked tensor): the
// estimate of its sum of U_hat^2, the estimate's absolute error bound, and whether its
// floor regime leaves the sum open (the estimate is then an upper bound). Records q and
// the next step's floor regime of the slice.
//
// Row-band tensors: when no element is on the eps floor (min R_i * min c'_j >= eps) the
// sum is sum_j z_j / c'_j, with a spread bounded through max (s x)^2 / (R_i c'_j); when
// every element is (max R_i * max c'_j < eps) it is the exactly rounded floored sum.
// Otherwise both are upper bounds of the oracle's sum (an element's U_hat^2 is at most
// its unfloored and its floored value, up to rounding).
struct SliceSum {
  double S, E;
  int open;     // 0, or why the sum is open (kWhyStraddle, kWhyMissingSum)
  int bad;      // a non-finite sum or statistic
  int repeats;  // the R_i or the c'_j repeat: the spread of the fast sum is not statistical
};

// The spread bounds of the fast sums take the roundings of R_i c'_j, of the square root and
// of the quotient as independent from element to element. When the R_i or the C_j of a
// factored tensor repeat (all equal, as under a constant gradient, or many equal neighbours,
// as under a gradient of a few distinct magnitudes), the first two roundings repeat with
// them and do not average out. Such a tensor takes the rigorous bound instead: each term of
// the fast sum lies within 5.05 u (u = 2^-24) of the oracle's rounded U_hat^2.
constexpr double kRigorousRel = 5.05 * 0x1p-24;
// all (nearly) equal, or more than 1/64 of neighbours equal (never seen with gradients of
// continuous distribution: R_i and C_j are sums of many squares); the extremes are over
// positive values (of R and C, or of R and c' = C / q: the same ratio)
__device__ __forceinline__ int repeats_rule(const DevTensor &t, float rmn, float rmx, float cmn, float cmx,
                                            double dup_r, double dup_c) {
  const bool ur = t.n > 1 && rmx <= rmn * (1.f + 0x1p-20f);
  const bool uc = t.m > 1 && cmx <= cmn * (1.f + 0x1p-20f);
  return (ur || uc || 64.0 * dup_r > (double)t.n || 64.0 * dup_c > (double)t.m) ? 1 : 0;
}

template <class Red>
__device__ __forceinline__ SliceSum slice_sum(const DevTensor &t, const StepConsts &k, const Red &r) {
  SliceSum o = {0.0, 0.0, 0, 0, 0};
  const bool factored = t.kind == kFactored;
  // s: the sum of R (wide factored tensors), then of the row-band tensors Y, S and S2 (below), of
  // others the sum of U_hat^2, nothing and the sum of U_hat^4; and the repeats of R and of C
  RedAll a;
  if (factored && !t.zpath && Red::kN == kThreads) a.s[0] = sum_r_part(t, k, r.lane());
  if (t.zpath) {
    for (int64_t b = r.lane(); b < t.nzb; b += Red::kN) {
      const BandStats *x = t.bst + b;
      a.s[1] += ldg(&x->ysum);
      a.um = fmax(a.um, ldg(&x->umax));
      a.rmn = fminf(a.rmn, ldg(&x->rmin));
      a.rmx = fmaxf(a.rmx, ldg(&x->rmax));
      a.bad |= ldg(&x->bad);
      a.s[4] += (double)ldg(&x->rdup);
    }
    for (int64_t c = r.lane(); c < t.nfc; c += Red::kN) {
      const ColStats *x = t.cst + c;
      a.s[2] += ldg(&x->s);
      a.s[3] += ldg(&x->s2);
      a.cmn = fminf(a.cmn, ldg(&x->cmin));
      a.cmx = fmaxf(a.cmx, ldg(&x->cmax));
      a.bad |= ldg(&x->bad);
      a.s[5] += (double)ldg(&x->cdup);
    }
  } else {
    if (factored)   // the fold's per-chunk statistics of R and C
      for (int64_t q = r.lane(); q < (int64_t)t.nfr + t.nfc; q += Red::kN) {
        const ColStats *c = t.cst + q;
        const float mn = ldg(&c->cmin), mx = ldg(&c->cmax);
        const double d = (double)ldg(&c->cdup);
        if (q < t.nfr) {
          a.rmn = fminf(a.rmn, mn);
          a.rmx = fmaxf(a.rmx, mx);
          a.s[4] += d;
        } else {
          a.cmn = fminf(a.cmn, mn);
          a.cmx = fmaxf(a.cmx, mx);
          a.s[5] += d;
        }
      }
    const int64_t ntiles = (int64_t)t.ntr * t.ntc * kSub;   // per-part sums
    for (int64_t c = r.lane(); c < ntiles; c += Red::kN) {
      a.s[1] += ldg(t.ssum + c);
      a.s[3] += ldg(t.qsum + c);
    }
  }
  r.all(a);
  // (the fold has formed a row-band tensor's q)
  const float q = !factored || t.zpath ? 0.f : mean_r_from(t, k, Red::kN == kThreads ? a.s[0] : sum_r_wave(t, k));
  if (factored) o.repeats = repeats_rule(t, a.rmn, a.rmx, a.cmn, a.cmx, a.s[4], a.s[5]);
  if (t.zpath) {
    // SU2: the sum over the terms t_ij = (s x)^2 / (R_i c'_j) of t_ij^2 <= umax * sum_j z_j / c'_j^2
    const double Y = a.s[1], SU = a.s[2], SU2 = a.s[3], um = a.um;
    const float rmn = a.rmn, rmx = a.rmx, cmn = a.cmn, cmx = a.cmx;
    const int bad = a.bad;
    // the sums the row-band pass formed this step (it skips one when the last step
    // predicts the regime); a sum it did not form counts as +inf
    const int formed = ldg(&t.bst[0].regime);
    const bool have_z = formed != kRegimeFloor, have_y = formed != kRegimeAbove;
    const double inf = __builtin_inf();
    const double SUf = have_z ? SU : inf, Yf = have_y ? Y : inf;
    const bool finite = !(SUf != SUf) && !(Yf != Yf) && (SUf < 1e300 || Yf < 1e300);
    const float lo = __fmul_rn(rmn, cmn), hi = __fmul_rn(rmx, cmx);
    if (bad || !finite) {
      o.bad = 1;
      o.S = SU;
    } else if (have_z && lo >= k.eps) {   // nothing on the floor
      o.S = SU;
      o.E = SU > 0.0 ? 20.0 * 0x1p-23 * sqrt(um * SU2) + 1e-14 * SU : 0.0;
      if (o.repeats) o.E = fmax(o.E, kRigorousRel * SU + 1e-14 * SU);
    } else if (have_y && hi < k.eps) {    // everything on the floor
      o.S = Y;
      o.E = 1e-14 * Y;
    } else {
      o.S = fmin(SUf, Yf) * (1.0 + 1e-6);  // an upper bound of the oracle's sum
      o.open = (have_z && have_y) ? kWhyStraddle : kWhyMissingSum;
    }
    // the next step's prediction. Without new gradient R_i c'_j only decays by beta2 per
    // step, but a larger gradient can lift it by any factor: a 5% margin above the floor,
    // a factor 2 below it. A wrong prediction costs a re-check at most.
    const int next = (lo >= 1.05f * k.eps) ? kRegimeAbove : (2.f * hi < k.eps ? kRegimeFloor : kRegimeBoth);
    if (r.lead()) stg(&t.sc->regime, o.bad ? (int32_t)kRegimeBoth : (int32_t)next);
  } else {
    o.S = a.s[1];
    const double Q4 = a.s[3];
    // the exact second moment's sum is the oracle's own; a factored one carries the
    // spread of its unrounded terms (20 standard deviations)
    o.E = t.kind == kFactored ? 20.0 * 0x1p-23 * sqrt(Q4) + 1e-14 * o.S : 0.0;
    if (o.repeats) o.E = fmax(o.E, kRigorousRel * o.S + 1e-14 * o.S);
  }
  if (!t.zpath && r.lead()) stg(&t.sc->q, q);
  return o;
}

// The clip stage's share of each slice of the stacked tensors, one wave per slice: its fast
// sum, error bound and flags (kept in its scalars for the group's decision and, should the
// stack's sum be open, for its re-check), its q and its next regime.
__global__ __launch_bounds__(kThreads) void clip_slices_kernel(const DevTensor *__restrict__ TT,
                                                               const Item *__restrict__ items, int64_t count,
                                                               StepConsts k) {
  const int64_t j = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
  if (j >= count) return;   // a whole wave
  const DevTensor &t = TT[items[j].tensor];
  const SliceSum o = slice_sum(t, k, RedWave{});
  if ((threadIdx.x & 63) == 0) {
    stg(&t.sc->s_fast, o.S);
    stg(&t.sc->e_fast, o.E);
    stg(&t.sc->fast_flags, (int32_t)((o.open & 15) | (o.bad ? 16 : 0) | (o.repeats ? 32 : 0)));
  }
}

// --------------------------------------------------------------------------------------------
// clip stage, one work-group per tensor (or per stacked tensor, whose slices share one k):
// k = 1 / max(1, RMS(U_hat) / d) (Sec. 3, Alg. 1), NaN-propagating and rounded once to
// float as the oracle rounds it. It records q = max(mean R, eps) and flags the tensor when
// k's rounding is not decided by the approximate sum: its spread (20 standard deviations
// of the free roundings) reaches a rounding boundary of k or the clipping threshold. When
// a slice's floor regime leaves its sum open, the group's sum is an upper bound: below
// the clipping threshold k is exactly 1, and above it the tensor goes to a re-check.
// --------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void clip_kernel(const DevTensor *__restrict__ TT,
                                                        const Item *__restrict__ items, StepConsts k,
                                                        RecheckLists *L, int ntensors) {
  __shared__ double sh[kThreads];
  __shared__ double wsum[kWaves][3];
  __shared__ int wflag[kWaves][4];
  __shared__ float kf_sh;
  __shared__ int st_sh, pos_sh;
  // a stack's open slices, for a floor-split re-check of those alone (stacks of up to
  // kOpenBits slices; a larger one re-reads every slice)
  constexpr int kOpenBits = 32 * 64;
  __shared__ uint32_t openbits[kOpenBits / 32];
  const Item it = items[blockIdx.x];   // the first sub-tensor of a group sharing one k
  const DevTensor &t0 = TT[it.tensor];
  const int g0 = t0.grp0, ng = t0.ngrp;
  // the group's sum S as the sum of its slices' estimates, with the sum of their absolute
  // error bounds, in slice order within a wave and then wave by wave
  double S = 0.0, err = 0.0, N = 0.0;
  int open = 0;   // why the first open slice (in slice order) is open
  bool bad_any = false, rep_any = false;
  if (ng == 1) {
    const SliceSum o = slice_sum(t0, k, RedGroup{sh});
    S = o.S;
    err = o.E;
    N = (double)(t0.n * t0.m);
    open = o.open;
    bad_any = o.bad != 0;
    rep_any = o.repeats != 0;
  } else {
    // the slices' sums come from clip_slices_kernel (launched just before)
    for (int q = (int)threadIdx.x; q < kOpenBits / 32; q += kThreads) openbits[q] = 0u;
    __syncthreads();
    const int w = (int)(threadIdx.x >> 6);
    double s = 0.0, e_ = 0.0, nn = 0.0;
    int first = 0x7fffffff, why = 0, bad = 0, rep = 0;   // the wave's first open slice, and why it is open
    for (int e = w; e < ng; e += kWaves) {
      const DevTensor &t = TT[g0 + e];
      const int fl = ldg(&t.sc->fast_flags);
      const SliceSum o = {ldg(&t.sc->s_fast), ldg(&t.sc->e_fast), fl & 15, (fl >> 4) & 1, (fl >> 5) & 1};
      if ((threadIdx.x & 63) == 0 && o.open && e < kOpenBits) atomicOr(&openbits[e >> 5], 1u << (e & 31));
      s += o.S;
      e_ += o.E;
      nn += (double)(t.n * t.m);
      if (o.open && first == 0x7fffffff) {
        first = e;
        why = o.open;
      }
      bad |= o.bad;
      rep |= o.repeats;
    }
    if ((threadIdx.x & 63) == 0) {
      wsum[w][0] = s;
      wsum[w][1] = e_;
      wsum[w][2] = nn;
      wflag[w][0] = first;
      wflag[w][1] = why;
      wflag[w][2] = bad;
      wflag[w][3] = rep;
    }
    __syncthreads();
    int f = 0x7fffffff;
    for (int v = 0; v < kWaves; v++) {   // waves in order
      S += wsum[v][0];
      err += wsum[v][1];
      N += wsum[v][2];
      if (wflag[v][0] < f) {
        f = wflag[v][0];
        open = wflag[v][1];
      }
      bad_any |= wflag[v][2] != 0;
      rep_any |= wflag[v][3] != 0;
    }
  }
  if (threadIdx.x == 0) {
    bool amb = (k.flags & SKEW_FLAG_EXACT_CLIP) != 0 && t0.kind == kFactored;
    int why = amb ? kWhyForced : (open ? open : 0);
    int level = 2;   // the re-check a flagged group gets
    double spread = 0.0;
    if (bad_any) {
      amb = true;
      why = kWhyNonFinite;
    } else if (open) {
      S += err;   // an upper bound of the group's sum
      if (!(sqrt(S / N) / (double)k.d < 1.0) && !amb) {
        amb = true;
        // the floor split per element decides most of these, except where the factors
        // repeat (its spread is statistical too). A tensor whose terms left the split's
        // spread wide (heavy tails) keeps them from step to step: when the last split's
        // relative spread makes an undecided k likely (more than 0.55 of the spacing of k's
        // floats near the estimate: the exact sequence costs about 1/0.45 of the split's
        // vector work), it goes straight to the exact sequence. Every eighth step takes
        // the split, which renews the spread. The choice only saves a pass.
        const double r = sqrt(S / N) / (double)k.d;
        const float kg = (float)(1.0 / r);
        const double gap = (double)nextafterf(kg, 3.0e38f) - (double)kg;
        const bool wide = (double)ldg(&t0.sc->split_spread) * (1.0 / r) > 0.55 * gap && (k.step & 7) != 0;
        level = (rep_any || wide) ? 2 : 1;
      }
    } else {
      spread = S > 0.0 ? err / S : 0.0;
    }
    const bool flagged_before = amb;
    kf_sh = clip_from_sum(S, N, k.d, spread, amb);
    if (amb && !flagged_before) why = kWhySpread;
    const bool list = amb && t0.kind == kFactored;
    pos_sh = list ? atomicAdd(level == 1 ? &L->n1 : &L->n2, ng) : 0;
    st_sh = list ? (int)((level == 1 ? kClipPending1 : kClipPending2) | (why << 4)) | (level << 16) : -1;
  }
  __syncthreads();
  const float kf = kf_sh;
  const int st = st_sh, pos = pos_sh;
  // a stack's floor-split re-check reads its first slice (whose work-group decides k) and
  // its open slices; the others are listed as -1 and keep their fast sums
  const bool partial = (st >> 16) == 1 && ng > 1 && ng <= kOpenBits;
  for (int e = (int)threadIdx.x; e < ng; e += kThreads) {
    const DevTensor &t = TT[g0 + e];
    stg(&t.sc->k, kf);
    if (st >= 0) {
      const bool keep = partial && e > 0 && !((openbits[e >> 5] >> (e & 31)) & 1u);
      stg(recheck_list(L, ntensors, st >> 16) + pos + e, keep ? (int32_t)-1 : (int32_t)(g0 + e));
      stg(&t.sc->ambiguous, (int32_t)(st & 0xFFFF));
    } else {
      stg(&t.sc->ambiguous, (int32_t)kClipFast);
    }
  }
}

// The weight the update starts from: w - (lr lambda) w with one rounding when the decoupled
// weight decay applies (Sec. 3 footnote, Sec. 6), else w itself
__device__ __forceinline__ float decayed(float w, bool dec, float wd) { return dec ? fmaf(-wd, w, w) : w; }

// The oracle's float sequence for one factored element (Alg. 1 with the eps clamps):
// D = sqrt(max(R_i * c'_j, eps)), U = ((s * x) / D) * k, y = (wd - lr U) + xi, where wd is
// the (decayed) starting weight and xi scales with the pre-step |w|.
__device__ __forceinline__ float exact_factored_y(float x, float w, float wd, float Ri, float cpj, float s,
                                                  float kc, float eps, float lr, float dith, bool xu) {
  const float vh = __fmul_rn(Ri, cpj);
  const float dd = sqrtf(max_nan(vh, eps));
  const float U = __fmul_rn(__fmul_rn(s, x) / dd, kc);
  return fmaf(dith, dither_mul(w, xu), fmaf(-lr, U, wd));
}

// y may round differently from the oracle's value when this is >= 0: the fast update x*F
// differs from the oracle's lr*U by < 2^-19 relative, and each of x and y carries one
// rounding. (y - mid is exact and finite for finite y; NaN never counts as near.)
__device__ __forceinline__ float boundary_slack(float y, float xF, float w) {
  // the midpoint between y's two bf16 neighbours: y's high half, then 0x8000
  const float mid = __uint_as_float(__builtin_amdgcn_perm(__float_as_uint(y), 0x8000u, 0x07060100u));
  const float bound = fmaf(fabsf(xF), 0x1p-18f + 0x1p-21f, fabsf(w) * 0x1p-21f);
  return bound - fabsf(y - mid);
}
__device__ __forceinline__ bool near_boundary(float y, float xF, float w) { return boundary_slack(y, xF, w) >= 0.f; }

struct P3Scalars {
  float q, s, kc, cap3, eps, lr, gc;
  double lsk;
};

// How a factored tensor's rows lie: aligned multiples of 8 columns (kPacked: taken several at a
// time); at any position, of 8 columns or more; of fewer
enum { kAligned = 0, kRagged = 1, kNarrow = 2, kPacked = 3 };
// kRagged: the lane at a row's end works on the row's last 8 elements (p on), of which the lane
// before it owns the first `over`: it computes them too (from values that may be new already) and
// stores its own only. Rows of fewer than 8 start at their first column.
// A template argument tells the two apart: with a branch at each load (whose result the branches
// share) every load would be waited for before the next went out.
template <int RAG>
__device__ __forceinline__ u32x4_t load8_from(const uint16_t *p, const Cols8 &c) {
  return RAG == kNarrow ? load8(p, c) : ldg_u_nt(p);
}
template <int RAG>
__device__ __forceinline__ void load8_from(const float *p, const Cols8 &c, float *o) {
  if constexpr (RAG == kNarrow) {
    load8(p, c, o);
  } else {
    const u32x4_t a = ldg_u(p), b = ldg_u(p + 4);
#pragma unroll
    for (int e = 0; e < 4; e++) {
      o[e] = __uint_as_float(a[e]);
      o[4 + e] = __uint_as_float(b[e]);
    }
  }
}
__device__ __forceinline__ void store8_from(uint16_t *p, const Cols8 &c, const uint4 &v) {
  u32x4_t o = {v.x, v.y, v.z, v.w};
  if (c.over != 0 && !c.narrow) shift_down(o, c.over);
  store8(p, c, to_uint4(o));
}
__device__ __forceinline__ void store8_from(float *p, const Cols8 &c, const float *v) {
  if (c.over != 0 && !c.narrow) {
    u32x4_t a, b;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      a[e] = __float_as_uint(v[e]);
      b[e] = __float_as_uint(v[4 + e]);
    }
    shift_down(a, b, c.over);
    float o[8];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      o[e] = __uint_as_float(a[e]);
      o[4 + e] = __uint_as_float(b[e]);
    }
    store8(p, c, o);
  } else {
    store8(p, c, v);
  }
}

// one row segment of 8 elements: momentum, update, dither, bf16 store. The fast path forms 1/D
// from per-row and per-column factors; the few elements whose result might round to the other
// bf16 neighbour take the oracle's exact sequence. RAG: the row may start at any position and
// end within the 8 columns.
template <bool XU, bool DEC, bool GC, int RAG>
__device__ __forceinline__ void p3_row8(const DevTensor &t, const StepConsts &k, const P3Scalars &c,
                                        const Dither &dz, const LaneMap &lm, int64_t i, int64_t wi, int64_t mi,
                                        const float *bf, uint4 gw, uint4 ww, const float *mv) {
  const bool mom = t.momentum != 0;
  // i: the block's first row (uniform; the lane's row is i + sub), wi and mi: the chunk's first
  // element of that row in W and in M
  const Cols8 cols(lm.over, RAG == kNarrow);
  const uint32_t om = (uint32_t)(lm.sub * (int)t.m + lm.col);   // (sub > 0 only where this fits)
  float x[8], w[8];
  unpack8(gw, x);
  unpack8(ww, w);
  if (GC) {
#pragma unroll
    for (int e = 0; e < 8; e++) x[e] = c.gc * x[e];
  }
  if (mom) {
#pragma unroll
    for (int e = 0; e < 8; e++) x[e] = fmaf(k.a1, x[e], __fmul_rn(k.b1, mv[e]));
    if constexpr (RAG == kRagged || RAG == kNarrow)
      store8_from(t.M + mi + (int)om, cols, x);
    else
      store_m8(t.M + mi + om, x);
  }
  const float alpha = (float)(c.lsk * ldg(t.ainv + i + lm.sub));
  // pair indices reach 2^32 only in tensors of more than 2^33 elements (a uniform test)
  const bool wide = t.idx0 + t.n * t.m > (int64_t(1) << 33);
  const uint64_t idx = (uint64_t)(t.idx0 + mi + ((RAG == kRagged || RAG == kNarrow) ? (int64_t)(int)om : (int64_t)om));
  float y[8], dith[8];
  if constexpr (RAG == kRagged || RAG == kNarrow) {
    dither8(dz, idx, wide, dith);
  } else {
    // pairs p0 .. p0 + 3: m and col are multiples of 8, so p0 is a multiple of 4 and the
    // four pairs share their high word and differ only in the low two bits
    const uint64_t p0 = idx >> 1;
    const uint32_t base = wide ? dz.pair_base(p0) : ((uint32_t)p0 ^ dz.klo ^ dz.inner0);
#pragma unroll
    for (int e2 = 0; e2 < 4; e2++) {
      const uint32_t h = fmix32(base ^ (uint32_t)e2);
      dith[2 * e2] = dither_lo(h);
      dith[2 * e2 + 1] = dither_hi(h);
    }
  }
  const bool dec = DEC && t.decay;
  constexpr bool xu = XU;
  float slack = -1.f;
#pragma unroll
  for (int e = 0; e < 8; e++) {
    const float F = fminf(alpha * bf[e], c.cap3);
    y[e] = fmaf(dith[e], dither_mul(w[e], xu), fmaf(-x[e], F, decayed(w[e], dec, k.wd)));
    slack = fmaxf(slack, boundary_slack(y[e], x[e] * F, w[e]));
  }
  if (slack >= 0.f) {
    const float Ri = ldg(t.R + i + lm.sub);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const float F = fminf(alpha * bf[e], c.cap3);
      if ((RAG != kNarrow || e < cols.count()) && near_boundary(y[e], x[e] * F, w[e]))
        y[e] = exact_factored_y(x[e], w[e], decayed(w[e], dec, k.wd), Ri, ldg(t.C + lm.c0 + lm.col + e) / c.q, c.s, c.kc,
                                c.eps, c.lr, dith[e], xu);
    }
  }
  const uint4 out = make_uint4(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]),
                               pack_bf16x2(y[6], y[7]));
  if constexpr (RAG == kRagged || RAG == kNarrow)
    store8_from(t.w + wi + (lm.sub * (int)t.ld + lm.col), cols, out);
  else
    stg_nt(reinterpret_cast<uint4 *>(t.w + wi + (uint32_t)(lm.sub * (int)t.ld + lm.col)), out);
}

template <bool XU, bool DEC, bool GC, int RAG>
__device__ __forceinline__ void p3_factored(const DevTensor &t, const Tile &tl, const StepConsts &k, float kc,
                                            float q, const Dither &dz) {
  const LaneMap lm(t, tl, RAG != kAligned && LaneMap::packs(t, tl));
  const int64_t n = t.n, m = t.m, ld = t.ld;
  const bool mom = t.momentum != 0;
  if (lm.idle) return;
  const Cols8 cols(lm.over, RAG == kNarrow);
  P3Scalars c;
  c.q = q;
  c.s = mom ? k.s_m : k.s_0;
  c.kc = kc;
  c.eps = k.eps;
  c.lr = k.lr;
  c.lsk = (double)k.lr * (double)c.s * (double)kc;   // lr * s * k
  c.gc = GC ? ldg(k.gscale) : 1.f;             // gradient-norm mode: elements are fl(c g)
  c.cap3 = (float)(c.lsk / (double)sqrtf(k.eps));
  float bf[8];
#pragma unroll
  for (int e = 0; e < 8; e++) bf[e] = RAG != kNarrow || e < cols.count() ? (float)col_factor(t, lm.c0 + lm.col + e, c.q) : 0.f;
  const int og = lm.sub * (int)ld + lm.col, om = lm.sub * (int)m + lm.col;   // (sub > 0 only where these fit)
  // (uniform offsets, stepped: 64-bit products in the loop delay its loads. The ragged path has no
  // registers left for the steps: it spills with them, and ran 2.5% slower)
  constexpr bool kStep = RAG == kAligned || RAG == kPacked;
  const int64_t dg = kStep ? lm.step * ld : 0, dm = kStep ? lm.step * m : 0;
  int64_t gi = lm.row * ld + lm.c0, mi = lm.row * m + lm.c0;
  for (int64_t i = lm.row; i + lm.sub < n; i += 2 * lm.step, gi += 2 * dg, mi += 2 * dm) {
    if constexpr (!kStep) {
      gi = i * ld + lm.c0;
      mi = i * m + lm.c0;
    }
    // the second row, where there is one; lanes without one load a row of their wave's again
    const bool more = i + lm.step < n, two = i + lm.step + lm.sub < n;
    const int og2 = two || !more ? og : lm.col, om2 = two || !more ? om : lm.col;
    const int64_t gi2 = more ? (kStep ? gi + dg : (i + lm.step) * ld + lm.c0) : gi;
    const int64_t mi2 = more ? (kStep ? mi + dm : (i + lm.step) * m + lm.c0) : mi;
    uint4 ga, wa, gb, wb;
    float ma[8], mb[8];
    if constexpr (RAG == kRagged || RAG == kNarrow) {
      ga = to_uint4(load8_from<RAG>(t.g + gi + og, cols));
      wa = to_uint4(load8_from<RAG>(t.w + gi + og, cols));
      gb = to_uint4(load8_from<RAG>(t.g + gi2 + og2, cols));
      wb = to_uint4(load8_from<RAG>(t.w + gi2 + og2, cols));
    } else {
      ga = ldg_nt(reinterpret_cast<const uint4 *>(t.g + gi + (uint32_t)og));
      wa = ldg_nt(reinterpret_cast<const uint4 *>(t.w + gi + (uint32_t)og));
      gb = ldg_nt(reinterpret_cast<const uint4 *>(t.g + gi2 + (uint32_t)og2));
      wb = ldg_nt(reinterpret_cast<const uint4 *>(t.w + gi2 + (uint32_t)og2));
    }
    if (mom) {
      if constexpr (RAG == kRagged || RAG == kNarrow) {
        load8_from<RAG>(t.M + mi + om, cols, ma);
        load8_from<RAG>(t.M + mi2 + om2, cols, mb);
      } else {
        load_m8(t.M + mi + (uint32_t)om, ma);
        load_m8(t.M + mi2 + (uint32_t)om2, mb);
      }
    }
    p3_row8<XU, DEC, GC, RAG>(t, k, c, dz, lm, i, gi, mi, bf, ga, wa, ma);
    if (two) p3_row8<XU, DEC, GC, RAG>(t, k, c, dz, lm, i + lm.step, gi2, mi2, bf, gb, wb, mb);
  }
}

template <bool XU, bool DEC, bool GC>
__device__ __forceinline__ void p3_exact(const DevTensor &t, const Tile &tl, const StepConsts &k, float kc,
                                         const Dither &dz) {
  // exact second moment: the oracle's operation order exactly
  const WaveMap wm(t, tl);
  const int64_t m = t.m, ld = t.ld, col = wm.col;
  const bool mom = t.momentum != 0;
  if (col >= m) return;
  const Cols8 cols(m, col);
  const float gc = GC ? ldg(k.gscale) : 1.f;
  const bool wide = t.idx0 + t.n * t.m > (int64_t(1) << 33);
  constexpr bool xu = XU;
  for (int64_t lr = wm.wr; lr < tl.nr; lr += wm.rpi) {
    const int64_t i = tl.row(lr);
    float g[8], w[8], v[8], mo[8];
    load_elems8(t.g, i * ld, cols, t.fp32, g);
    load_elems8(t.w, i * ld, cols, t.fp32, w);
    load8(t.V + i * m, cols, v);
    if (mom) load8(t.M + i * m, cols, mo);
    float dith[8];
    if (!t.fp32) dither8(dz, (uint64_t)t.idx0 + (uint64_t)i * (uint64_t)m + (uint64_t)col, wide, dith);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      if (GC) g[e] = gc * g[e];
      v[e] = fmaf(k.a2, __fmul_rn(g[e], g[e]), __fmul_rn(k.b2, v[e]));
      const float dd = sqrtf(max_nan(v[e], k.eps));
      float num;
      if (mom) {
        mo[e] = fmaf(k.a1, g[e], __fmul_rn(k.b1, mo[e]));
        num = __fmul_rn(k.s_m, mo[e]);
      } else {
        num = __fmul_rn(k.s_0, g[e]);
      }
      const float U = __fmul_rn(num / dd, kc);
      const float x = fmaf(-k.lr, U, decayed(w[e], DEC && t.decay, k.wd));
      // (float32 masters: no dither, no cast)
      w[e] = t.fp32 ? x : fmaf(dith[e], dither_mul(w[e], xu), x);
    }
    store8(t.V + i * m, cols, v);
    if (mom) store8(t.M + i * m, cols, mo);
    if (t.fp32)
      store8(reinterpret_cast<float *>(t.w) + i * ld, cols, w);
    else
      store8(t.w + i * ld, cols, make_uint4(pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3]),
                                            pack_bf16x2(w[4], w[5]), pack_bf16x2(w[6], w[7])));
  }
}

// --------------------------------------------------------------------------------------------
// p3: clip factor, state update, weight update and dithered bf16 write-back (Alg. 1)
// --------------------------------------------------------------------------------------------
// XU: the exact-ulp dither; DEC: the decoupled weight decay is on (lr lambda != 0); GC: the
// gradient-norm mode (elements enter as fl(c g)); RAG: the table has a factored tensor whose rows
// are not all 16-byte aligned multiples of 8 columns (its path takes registers from the other:
// with both in every instantiation the 6.78B-like tables' pass ran 1.5% slower)
// (at most 128 VGPRs: four waves per SIMD keep enough loads in flight)
template <bool XU, bool DEC, bool GC, bool RAG>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void p3_kernel(const DevTensor *__restrict__ TT,
                                                      const Item *__restrict__ items, StepConsts k,
                                                      RecheckLists *L) {
  // the re-check lists of this step are consumed: empty them for the next
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    stg(&L->n1, 0);
    stg(&L->n2, 0);
  }
  const Item it = items[blockIdx.x];
  const DevTensor &t = TT[it.tensor];
  const Tile tl = tile_of(t, it.tile);
  const float kc = ldg(&t.sc->k);
  const Dither dz(k.seed, k.step, t.tensor_id);
  if (t.kind == kFactored) {
    if (!RAG || t.vec) {
      if (LaneMap::packs(t, tl))
        p3_factored<XU, DEC, GC, kPacked>(t, tl, k, kc, ldg(&t.sc->q), dz);
      else
        p3_factored<XU, DEC, GC, kAligned>(t, tl, k, kc, ldg(&t.sc->q), dz);
    } else if constexpr (RAG) {
      if (t.m < 8)
        p3_factored<XU, DEC, GC, kNarrow>(t, tl, k, kc, ldg(&t.sc->q), dz);
      else
        p3_factored<XU, DEC, GC, kRagged>(t, tl, k, kc, ldg(&t.sc->q), dz);
    }
  } else
    p3_exact<XU, DEC, GC>(t, tl, k, kc, dz);
}

}  // namespace

// The static workspace of skew_state_init_static: device memory the library itself holds
// on every GPU it runs on, for callers that cannot allocate. Host code never passes the
// array's name to a kernel or a copy: it takes the array's device address on each device
// from hipGetSymbolAddress (looked up once per device, with that device current).
static __device__ __align__(256) unsigned char scratch[SKEW_STATIC_WORKSPACE_BYTES];

int static_workspace(void **ptr) {
  constexpr int kMaxDev = 64;
  static std::mutex mu;
  static void *addr[kMaxDev] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= kMaxDev) return (int)hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (addr[dev] == nullptr) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return (int)hipSuccess;
}

int launch_p1(const DevTensor *T, const Item *items, int64_t count, void *stream) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(p1_kernel, dim3((uint32_t)count), dim3(kThreads), 0, (hipStream_t)stream, T, items);
  return (int)hipGetLastError();
}
int launch_p1z(const DevTensor *T, const Item *items, int64_t count, const StepConsts &k, int mode, void *stream) {
  if (count <= 0) return hipSuccess;
  const dim3 grid((uint32_t)count), block(kZThreads);
  auto *kern = mode == 0 ? p1z_kernel<0> : (mode == 1 ? p1z_kernel<1> : p1z_kernel<2>);
  hipLaunchKernelGGL(kern, grid, block, 0, (hipStream_t)stream, T, items, k);
  return (int)hipGetLastError();
}
int launch_fold(const DevTensor *T, const Item *items, int64_t count, const StepConsts &k, int phase, void *stream) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(fold_kernel, dim3((uint32_t)count), dim3(kFoldThreads), 0, (hipStream_t)stream, T, items, k, phase);
  return (int)hipGetLastError();
}
int launch_gsq(const DevTensor *T, const Item *items, int64_t count, void *stream) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(gsq_kernel, dim3((uint32_t)count), dim3(kThreads), 0, (hipStream_t)stream, T, items);
  return (int)hipGetLastError();
}
int launch_gnorm(const DevTensor *T, int ntensors, const StepConsts &k, void *stream) {
  if (ntensors <= 0) return hipSuccess;
  hipLaunchKernelGGL(gsum_kernel, dim3((uint32_t)ntensors), dim3(kThreads), 0, (hipStream_t)stream, T, k);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return (int)e;
  hipLaunchKernelGGL(gnorm_kernel, dim3(1), dim3(kThreads), 0, (hipStream_t)stream, ntensors, k);
  return (int)hipGetLastError();
}
int launch_p2(const DevTensor *T, const Item *items, int64_t count, const StepConsts &k, void *stream) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(p2_kernel, dim3((uint32_t)count), dim3(kThreads), 0, (hipStream_t)stream, T, items, k);
  return (int)hipGetLastError();
}
int launch_clip_slices(const DevTensor *T, const Item *items, int64_t count, const StepConsts &k, void *stream) {
  if (count <= 0) return hipSuccess;
  const int64_t groups = (count + kWaves - 1) / kWaves;
  hipLaunchKernelGGL(clip_slices_kernel, dim3((uint32_t)groups), dim3(kThreads), 0, (hipStream_t)stream, T, items,
                     count, k);
  return (int)hipGetLastError();
}
int launch_clip(const DevTensor *T, const Item *items, int64_t count, const StepConsts &k, RecheckLists *L,
                int ntensors, void *stream) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(clip_kernel, dim3((uint32_t)count), dim3(kThreads), 0, (hipStream_t)stream, T, items, k, L,
                     ntensors);
  return (int)hipGetLastError();
}
int launch_recheck(const DevTensor *T, RecheckLists *L, int ntensors, const StepConsts &k, int level, void *stream) {
  if (ntensors <= 0) return hipSuccess;
  hipLaunchKernelGGL(recheck_kernel, dim3(kRecheckGrid), dim3(kThreads), 0, (hipStream_t)stream, T, L, ntensors, k,
                     level);
  return (int)hipGetLastError();
}
int launch_clip_recheck(const DevTensor *T, RecheckLists *L, int ntensors, const StepConsts &k, int level,
                        void *stream) {
  if (ntensors <= 0) return hipSuccess;
  hipLaunchKernelGGL(clip_recheck_kernel, dim3((uint32_t)ntensors), dim3(kThreads), 0, (hipStream_t)stream, T, L,
                     ntensors, k, level);
  return (int)hipGetLastError();
}
int launch_p3(const DevTensor *T, const Item *items, int64_t count, const StepConsts &k, RecheckLists *L,
              void *stream) {
  if (count <= 0) return hipSuccess;
  const bool xu = (k.flags & SKEW_FLAG_EXACT_ULP) != 0, dec = k.wd != 0.f, gc = k.gclip != 0;
  auto pick = [&](auto x, auto d, auto g) {
    return k.ragged ? p3_kernel<decltype(x)::value, decltype(d)::value, decltype(g)::value, true>
                    : p3_kernel<decltype(x)::value, decltype(d)::value, decltype(g)::value, false>;
  };
  const std::true_type yes;
  const std::false_type no;
  auto *kern = xu ? (dec ? (gc ? pick(yes, yes, yes) : pick(yes, yes, no)) : (gc ? pick(yes, no, yes) : pick(yes, no, no)))
                  : (dec ? (gc ? pick(no, yes, yes) : pick(no, yes, no)) : (gc ? pick(no, no, yes) : pick(no, no, no)));
  hipLaunchKernelGGL(kern, dim3((uint32_t)count), dim3(kThreads), 0, (hipStream_t)stream, T, items, k, L);
  return (int)hipGetLastError();
}

}  // namespace skew
