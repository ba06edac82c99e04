// Device-side helpers shared by the gfx950 kernels: vector types, streaming loads and stores,
// wavefront reductions, the counter-based Gaussian generator and the one rounding order of the
// CECA combine.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "launch.h"

namespace ceca {

typedef float vf4 __attribute__((ext_vector_type(4)));
// Four columns as they lie in memory: rows of any pitch and base, whose groups are aligned to 4 bytes only (a
// 16-byte load or store of this chip needs no more).
typedef float vf4_mem __attribute__((ext_vector_type(4), aligned(4)));

template <typename V> struct InMemory;
template <> struct InMemory<vf4> { using T = vf4_mem; };
template <> struct InMemory<float> { using T = float; };

template <int VEC> struct VecOf;
template <> struct VecOf<4> { using T = vf4; };
template <> struct VecOf<1> { using T = float; };

// The column tile of this workgroup.  Workgroups go round-robin over the 8 XCDs, each with its own L2.  Where a row
// of a tile is narrower than a 128-byte line, neighbouring tiles should meet in one L2, and the tiles in flight
// should lie close together so that the DRAM pages of a row are opened once: runs of kXcdRun adjacent tiles go to
// one XCD, the next run to the next.  Measured with 64-byte rows (identity rounds, n = 1026): 500 us in plain
// order, 386 with one contiguous eighth of all tiles per XCD, 397 / 359 / 341 / 337 / 352 with runs of 2 / 8 / 16
// / 32 / 64 at a power-of-two pitch; 415, 288 and 308 / 303 / 304 / 307 / 301 at a pitch 128 bytes longer.
// Over the register-tile kernels, 600 to 4096 agents and three pitches (2^26 elements) runs of 16 are within 4 % of the
// better of both or ahead, mostly ahead of the contiguous eighth by 5 to 15 % at power-of-two pitches, and behind it by up to 7 %
// where rows of the tile are 16 or 32 bytes (4096 agents) or the pitch is none (fused rounds, n = 1100, d = 61,008: 266
// us against 256).
__device__ __forceinline__ int64_t tile_of_block(int32_t xcd_runs) {
  const uint32_t b = blockIdx.x;
  if (!xcd_runs) return b;
  const uint32_t xcd = b & 7, q = b >> 3;
  return (int64_t)((q / kXcdRun * 8 + xcd) * kXcdRun + q % kXcdRun);
}

// State rows are touched once per round: stream them past the caches (nontemporal loads and stores).
template <typename V> __device__ __forceinline__ V ld_stream(const float* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const typename InMemory<V>::T*>(p));
}
template <typename V> __device__ __forceinline__ void st_stream(float* p, V v) {
  __builtin_nontemporal_store(v, reinterpret_cast<typename InMemory<V>::T*>(p));
}
template <typename V> __device__ __forceinline__ V ld_plain(const float* p) {
  return *reinterpret_cast<const typename InMemory<V>::T*>(p);
}
template <typename V> __device__ __forceinline__ void st_plain(float* p, V v) {
  *reinterpret_cast<typename InMemory<V>::T*>(p) = v;
}

// Rows whose length is no multiple of four end in a group of 1 to 3 columns.  Its thread loads the row's last four columns
// instead, `back` columns further left (rows have at least four), moves its own to the front, zeros behind them, and
// stores its own one by one.
__device__ __forceinline__ vf4 own_columns(vf4 v, int back) {
  if (back & 1) v = vf4{v.y, v.z, v.w, 0.0f};
  if (back & 2) v = vf4{v.z, v.w, 0.0f, 0.0f};
  return v;
}
__device__ __forceinline__ float own_columns(float v, int) { return v; }
// The other way round: its own columns where they lie in the row's last four, zeros in front of them.
__device__ __forceinline__ vf4 last_columns(vf4 v, int back) {
  if (back & 1) v = vf4{0.0f, v.x, v.y, v.z};
  if (back & 2) v = vf4{0.0f, 0.0f, v.x, v.y};
  return v;
}
__device__ __forceinline__ float last_columns(float v, int) { return v; }
// What a lane read of a row, with zeros for columns that are not its own, when `left` columns of the row are left from its first one
// on (fewer than four: it read the row's last four; none: anything).  Times z = 0 an infinite one would be NaN.
__device__ __forceinline__ vf4 own_of_row(vf4 a, int left) {
  return vf4{left < 4 ? 0.0f : a.x, left < 3 ? 0.0f : a.y, left < 2 ? 0.0f : a.z, left < 1 ? 0.0f : a.w};
}
__device__ __forceinline__ float own_of_row(float a, int) { return a; }
__device__ __forceinline__ int columns_left(int64_t col, int64_t d) { return (int)min(d - col, (int64_t)1 << 20); }
// Whether some lane of the wavefront has a NaN among its numbers.
template <int CH> __device__ __forceinline__ bool some_nan(const float (&m)[CH]) {
  float s = m[0];                          // (infinities of both signs ask for nothing but a second look)
#pragma unroll
  for (int j = 1; j < CH; ++j) s += m[j];
  return __any(s != s);
}

// How a register-tile kernel's tile goes about memory (TileMemory).  WHOLE: rows of whole groups that are streamed, the instance without
// the instructions for anything else.
template <bool WHOLE, typename Args> __device__ __forceinline__ auto tile_of(const Args& M) {
  auto mem = M.mem;
  if (WHOLE) mem.cached_loads = mem.cached_stores = mem.short_cols = 0;
  return mem;
}
// That distance for the group at column col.
template <typename Args> __device__ __forceinline__ int columns_back(const Args& M, int64_t col) {
  return col == (M.ngroups - 1) * 4 ? M.mem.short_cols : 0;
}

// How far back the 16-byte group at column `col` of a row of d columns has to be loaded (0 unless it is the short last
// one).  ODD: the length is no multiple of four; kernels come without the short group's instructions too.
template <bool ODD> __device__ __forceinline__ int short_back(int64_t col, int64_t d) {
  return ODD && col + 4 > d ? (int)(col + 4 - d) : 0;
}
// A group of a row of the caller's: loaded and stored whatever its place in the row (p: its first column).
template <typename V> __device__ __forceinline__ V ld_own(const float* p, int back) { return own_columns(ld_plain<V>(p - back), back); }
__device__ __forceinline__ void store_short(float* q, vf4 v, int back) {
  q[0] = v.x;
  if (back < 3) q[1] = v.y;
  if (back < 2) q[2] = v.z;
}
__device__ __forceinline__ void store_short(float* q, float v, int) { *q = v; }
template <typename V> __device__ __forceinline__ void st_own(float* p, V v, int back) {
  if (back) store_short(p, v, back);
  else st_plain<V>(p, v);
}

// RT rows of a tile, `step` rows apart, into registers: x from p and, with a second pointer, c from pc, row by row.
// Rows past row `last` hold what it does or, on a RING, those from row 0 on.  (The compiler must neither merge the two
// kinds of access, which would drop the streaming, nor work all addresses out in front of the branch.)
template <bool RING> __device__ __forceinline__ int row_of(int i, int last) {
  return RING ? (i > last ? i - last - 1 : i) : min(i, last);
}
template <typename V, int RT, bool TWO = true, bool RING = false>
__device__ __forceinline__ void load_rows(V (&x)[RT], const float* p, int64_t ld, V (&c)[RT], const float* pc, int64_t ldc, int row, int step,
                                          int last, bool cached) {
  if (cached) {
    asm volatile("; cached" : "+v"(row));
#pragma unroll
    for (int k = 0; k < RT; ++k) {
      const int64_t i = row_of<RING>(row + k * step, last);
      x[k] = ld_plain<V>(p + i * ld);
      if (TWO) c[k] = ld_plain<V>(pc + i * ldc);
    }
    asm volatile("; cached");
  } else {
    asm volatile("; streamed" : "+v"(row));
#pragma unroll
    for (int k = 0; k < RT; ++k) {
      const int64_t i = row_of<RING>(row + k * step, last);
      x[k] = ld_stream<V>(p + i * ld);
      if (TWO) c[k] = ld_stream<V>(pc + i * ldc);
    }
  }
}
template <typename V, int RT, bool RING = false>
__device__ __forceinline__ void load_rows(V (&x)[RT], const float* p, int64_t ld, int row, int step, int last, bool cached) {
  load_rows<V, RT, false, RING>(x, p, ld, x, nullptr, 0, row, step, last, cached);
}
// The same rows out of registers, those up to `last`; a short group's own columns one by one.
// x at p and, unless py is null (the same for every thread), y at py, row by row: all of x's rows before the first of y's
// measured up to 5 % slower (n = 258, 2^26 elements, fused rounds: 250 against 238 us).
template <typename V, int RT>
__device__ __forceinline__ void store_rows(const V (&x)[RT], float* p, const V (&y)[RT], float* py, int64_t ld, int row, int step, int last,
                                           int back, bool cached) {
  if (back) {
#pragma unroll
    for (int k = 0; k < RT; ++k) {
      if (row + k * step <= last) {
        const int64_t at = (int64_t)(row + k * step) * ld;
        store_short(p + at, x[k], back);
        if (py) store_short(py + at, y[k], back);
      }
    }
  } else if (cached) {
    asm volatile("; cached" : "+v"(row));
#pragma unroll
    for (int k = 0; k < RT; ++k) {
      if (row + k * step <= last) {
        const int64_t at = (int64_t)(row + k * step) * ld;
        st_plain<V>(p + at, x[k]);
        if (py) st_plain<V>(py + at, y[k]);
      }
    }
  } else {
    asm volatile("; streamed" : "+v"(row));
#pragma unroll
    for (int k = 0; k < RT; ++k) {
      if (row + k * step <= last) {
        const int64_t at = (int64_t)(row + k * step) * ld;
        st_stream<V>(p + at, x[k]);
        if (py) st_stream<V>(py + at, y[k]);
      }
    }
  }
}
template <typename V, int RT>
__device__ __forceinline__ void store_rows(const V (&x)[RT], float* p, int64_t ld, int row, int step, int last, int back, bool cached) {
  store_rows<V, RT>(x, p, x, nullptr, ld, row, step, last, back, cached);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}
// v + (v of lane ^ XOR), all in the vector unit: a trip through the LDS pipe (swizzle, lane exchange) costs about a
// hundred cycles in the reductions' dependent chains.  Distances 1 and 2 are quad permutes, 4 is a shift by four
// lanes up for the even banks of a row of 16 and down for the odd ones, 8 a rotation of the row by half; 16 and 32
// swap rows or halves between two registers that both hold v: one ends up with the lower, the other with the upper
// one's value in both places, and their sum is the pair's sum.
template <int XOR>
__device__ __forceinline__ float xor_add(float v) {
  const int bits = __builtin_bit_cast(int, v);
  if constexpr (XOR == 16 || XOR == 32) {
    typedef unsigned int pair __attribute__((ext_vector_type(2)));
    const pair s = XOR == 16 ? __builtin_amdgcn_permlane16_swap(bits, bits, false, false)
                             : __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
  } else {
    int moved;
    if constexpr (XOR == 1) moved = __builtin_amdgcn_update_dpp(0, bits, 0xB1, 0xf, 0xf, false);        // quad_perm [1, 0, 3, 2]
    else if constexpr (XOR == 2) moved = __builtin_amdgcn_update_dpp(0, bits, 0x4E, 0xf, 0xf, false);   // quad_perm [2, 3, 0, 1]
    else if constexpr (XOR == 4) {
      moved = __builtin_amdgcn_update_dpp(0, bits, 0x104, 0xf, 0x5, false);                              // row_shl:4 into banks 0 and 2
      moved = __builtin_amdgcn_update_dpp(moved, bits, 0x114, 0xf, 0xa, false);                          // row_shr:4 into banks 1 and 3
    } else moved = __builtin_amdgcn_update_dpp(0, bits, 0x128, 0xf, 0xf, false);                        // row_ror:8
    return v + __builtin_bit_cast(float, moved);
  }
}
// One level of the halving butterfly below: every lane adds its partner's copy of each of the 2H values
// it still carries, then keeps the H values that belong to its side (`up`); with one value left (H = 0)
// both partners keep the pair sum.  At distances 32 and 16 a swap of halves or rows between the two values of a pair
// puts what a lane keeps and its partner's copy of it into the two registers at once.
template <int XOR, int H>
__device__ __forceinline__ void halve(float (&m)[16], bool up) {
  if constexpr (H >= 1 && XOR >= 16) {
    typedef unsigned int pair __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int k = 0; k < H; ++k) {
      const int a = __float_as_int(m[k]), b = __float_as_int(m[k + H]);
      const pair s = XOR == 16 ? __builtin_amdgcn_permlane16_swap(a, b, false, false)
                               : __builtin_amdgcn_permlane32_swap(a, b, false, false);
      m[k] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    }
  } else if constexpr (H >= 1) {
    float s[2 * H];
#pragma unroll
    for (int k = 0; k < 2 * H; ++k) s[k] = xor_add<XOR>(m[k]);
#pragma unroll
    for (int k = 0; k < H; ++k) m[k] = up ? s[k + H] : s[k];
  } else {
    m[0] = xor_add<XOR>(m[0]);
  }
}
// Sums N <= 16 per-lane values (N a power of two) across the 64 lanes of a wavefront.  Each level halves the number of
// values a lane carries while there is more than one; the levels with the most values are the cheapest ones (32 and
// 16: one swap and one addition for a pair, no selects).  37 instructions for 16 values, the same bits for a value
// whatever N is.  Returns the complete sum of value number `which`; true in `owner` on exactly one lane per value.
template <int N>
__device__ __forceinline__ float wave_sum_many(const float (&in)[N], int lane, int& which, bool& owner) {
  static_assert(N == 1 || N == 2 || N == 4 || N == 8 || N == 16, "N must be a power of two up to 16");
  float m[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) m[k] = in[k < N ? k : 0];
  halve<32, N / 2>(m, false);
  halve<16, N / 4>(m, false);
  halve<8, N / 8>(m, lane & 8);
  halve<2, N / 16>(m, lane & 2);
  which = (N >= 2 && (lane & 32) ? N / 2 : 0) + (N >= 4 && (lane & 16) ? N / 4 : 0) + (N >= 8 && (lane & 8) ? N / 8 : 0) +
          (N >= 16 && (lane & 2) ? 1 : 0);
  constexpr int kept = (N >= 2 ? 32 : 0) | (N >= 4 ? 16 : 0) | (N >= 8 ? 8 : 0) | (N >= 16 ? 2 : 0);
  owner = (lane & ~kept) == 0;
  return xor_add<4>(xor_add<1>(m[0]));
}

// The 32-bit word of lane ^ XOR (XOR a power of two below 64): quad permutes for 1 and 2, swizzles inside
// each half of the wavefront for 4, 8 and 16, a lane exchange for 32.
template <int XOR>
__device__ __forceinline__ int xor_lane(int bits) {
  if constexpr (XOR == 1) return __builtin_amdgcn_update_dpp(0, bits, 0xB1, 0xf, 0xf, false);        // quad_perm [1, 0, 3, 2]
  else if constexpr (XOR == 2) return __builtin_amdgcn_update_dpp(0, bits, 0x4E, 0xf, 0xf, false);   // quad_perm [2, 3, 0, 1]
  else if constexpr (XOR == 32) return __shfl_xor(bits, 32, 64);
  else return __builtin_amdgcn_ds_swizzle(bits, (XOR << 10) | 0x1f);                                  // xor mask, all lanes kept
}
// The double that lane ^ XOR holds.
template <int XOR>
__device__ __forceinline__ double xor_lane(double v) {
  const int lo = xor_lane<XOR>(__double2loint(v));
  const int hi = xor_lane<XOR>(__double2hiint(v));
  return __hiloint2double(hi, lo);
}
// One level of a halving butterfly over doubles: a lane and its partner (lane ^ XOR) both carry 2H
// values; the lane keeps H of them (the upper half if `up`, which is the lane's own XOR bit) and adds the
// partner's copies of those.  With one value left (H = 0) both partners keep the pair sum.  The sum a
// lane forms is its own value plus the partner's, and the partner adds the same two numbers, so partners
// agree bit for bit.
template <int XOR, int H, int N>
__device__ __forceinline__ void halve_d(double (&v)[N], bool up) {
  if constexpr (H >= 1) {
    static_assert(2 * H <= N, "halving more values than the lane carries");
#pragma unroll
    for (int k = 0; k < H; ++k) {
      const double give = up ? v[k] : v[k + H];         // the half this lane drops is the half its partner keeps
      const double keep = up ? v[k + H] : v[k];
      v[k] = keep + xor_lane<XOR>(give);
    }
  } else {
    v[0] = v[0] + xor_lane<XOR>(v[0]);
  }
}

__device__ __forceinline__ float dot_v(vf4 a, vf4 b) { return a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w; }
// (the product is rounded by itself: fused into the first addition of a wavefront sum in one kernel and not in
// another, the same margin would get different bits)
__device__ __forceinline__ float dot_v(float a, float b) {
#pragma clang fp contract(off)
  return a * b;
}

// ---------------------------------------------------------------------------------------------
// Counter-based Gaussian noise (definition in ceca.h): one 32-bit word per uniform, Box-Muller
// on column pairs.  Transcendentals use the hardware's log2 / sin / cos (arguments in turns).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t mix32(uint32_t h) {
  h ^= h >> 16; h *= 0x7feb352du;
  h ^= h >> 15; h *= 0x846ca68bu;
  h ^= h >> 16;
  return h;
}
struct NoiseKeys { uint32_t k0, k1; };
__device__ __forceinline__ NoiseKeys noise_keys(uint32_t seed, uint32_t k, uint32_t agent) {
  NoiseKeys nk;
  nk.k0 = mix32(mix32(seed + 0x9e3779b9u * k) ^ agent);
  nk.k1 = mix32(nk.k0 + 0x85ebca6bu);
  return nk;
}
// The noise is what bounds the fused iterations, so its instructions are counted: integer multiplies run at
// the full vector rate on gfx950 (32 against 34 T lane-operations/s for a three-operand fused multiply-add),
// the transcendental units at half of it, and every other instruction costs the same.  The words of a group
// of four columns therefore share the first two steps of the hash, the conversions keep no instruction that
// is not exact anyway, and std * eps reaches e by one fused multiply-add per column.
//
// First two steps of word(c): c ^ k0, then h ^= h >> 16.  Columns that differ in their low two bits only
// differ there in those bits only, because h >> 16 does not see them.
__device__ __forceinline__ uint32_t noise_head(uint32_t c, NoiseKeys nk) {
  const uint32_t h = c ^ nk.k0;
  return h ^ (h >> 16);
}
// The remaining steps; the upper 24 bits of the word.
__device__ __forceinline__ uint32_t noise_tail24(uint32_t head, NoiseKeys nk) {
  uint32_t h = head * 0x7feb352du;
  h ^= h >> 15; h += nk.k1; h *= 0x846ca68bu;
  return (h >> 8) ^ (h >> 24);                           // (h ^ (h >> 16)) >> 8
}
// std * radius and the angle (in turns) of a column pair from its two words.
__device__ __forceinline__ void noise_polar(uint32_t w1, uint32_t w2, float std, float& rad, float& turns) {
#pragma clang fp contract(off)
  const float u1 = __builtin_fmaf((float)w1, 0x1p-24f, 0x1p-24f);    // (w1 + 1) / 2^24 in (0, 1], exact in fp32
  turns = (float)w2 * 0x1p-24f;                          // [0, 1), exact in fp32
  // -2 ln u1 = (2 ln 2) (-log2 u1); the factor's root goes with std, which is the same for every column
  rad = (std * 1.1774100225154747f) * __builtin_amdgcn_sqrtf(-__builtin_amdgcn_logf(u1));
}
// e + std * eps of the group's columns
template <typename V> __device__ __forceinline__ V add_noise(V e, float std, int64_t col, NoiseKeys nk);
template <> __device__ __forceinline__ vf4 add_noise<vf4>(vf4 e, float std, int64_t col, NoiseKeys nk) {
  const uint32_t h = noise_head((uint32_t)col, nk);      // col is a multiple of 4 on this path
  float r0, t0, r1, t1;
  noise_polar(noise_tail24(h, nk), noise_tail24(h ^ 1u, nk), std, r0, t0);
  noise_polar(noise_tail24(h ^ 2u, nk), noise_tail24(h ^ 3u, nk), std, r1, t1);
  e.x = __builtin_fmaf(r0, __builtin_amdgcn_cosf(t0), e.x);
  e.y = __builtin_fmaf(r0, __builtin_amdgcn_sinf(t0), e.y);
  e.z = __builtin_fmaf(r1, __builtin_amdgcn_cosf(t1), e.z);
  e.w = __builtin_fmaf(r1, __builtin_amdgcn_sinf(t1), e.w);
  return e;
}
template <> __device__ __forceinline__ float add_noise<float>(float e, float std, int64_t col, NoiseKeys nk) {
  const uint32_t h = noise_head((uint32_t)col & ~1u, nk);
  float r, t;
  noise_polar(noise_tail24(h, nk), noise_tail24(h ^ 1u, nk), std, r, t);
  return __builtin_fmaf(r, (col & 1) ? __builtin_amdgcn_sinf(t) : __builtin_amdgcn_cosf(t), e);
}

// z - lr e, the half step: one fused multiply-add, the same wherever it is evaluated.
__device__ __forceinline__ float half_step(float z, float lr, float e) { return __builtin_fmaf(-lr, e, z); }
__device__ __forceinline__ vf4 half_step(vf4 z, float lr, vf4 e) {
  vf4 o;
  o.x = half_step(z.x, lr, e.x); o.y = half_step(z.y, lr, e.y);
  o.z = half_step(z.z, lr, e.z); o.w = half_step(z.w, lr, e.w);
  return o;
}

// A value that every lane shares, in a vector register.  On gfx950 the plain fp32 and integer instructions (add,
// multiply, fused multiply-add, xor, and, shift) issue about 1.7 times as fast when all their operands are vector
// registers or constants as with one scalar-register operand (57 against 35 T lane-operations/s for a fused
// multiply-add), so factors that a loop applies to many elements are worth a vector register each.
template <typename T> __device__ __forceinline__ T in_vgpr(T uniform) {
  static_assert(sizeof(T) == 4, "one register");
  T v;
  asm("v_mov_b32 %0, %1" : "=v"(v) : "s"(uniform));
  return v;
}

// LDS by its own 32-bit addresses, so that a kernel can keep one as an integer and let a constant distance ride in
// the load instruction.
__device__ __forceinline__ uint32_t lds_address(const void* shared) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)shared;
}
template <typename V> __device__ __forceinline__ V lds_load(uint32_t address) {
  return *(__attribute__((address_space(3))) const V*)(uintptr_t)address;
}
template <typename V> __device__ __forceinline__ void lds_store(uint32_t address, V v) {
  *(__attribute__((address_space(3))) V*)(uintptr_t)address = v;
}

// w * self + wp * msg, with one fixed rounding order wherever it is evaluated: the product with self is
// rounded, then the peer's term is added by a fused multiply-add.  In this order the result can replace
// self in its own register (multiply in place, accumulate in place): kernels that carry self across a loop
// need no copy per element and round.
__device__ __forceinline__ float combine(float w, float self, float wp, float msg) {
#pragma clang fp contract(off)
  const float t = w * self;
  return __builtin_fmaf(wp, msg, t);
}
__device__ __forceinline__ vf4 combine(float w, vf4 self, float wp, vf4 msg) {
  vf4 o;
  o.x = combine(w, self.x, wp, msg.x); o.y = combine(w, self.y, wp, msg.y);
  o.z = combine(w, self.z, wp, msg.z); o.w = combine(w, self.w, wp, msg.w);
  return o;
}

}  // namespace ceca
