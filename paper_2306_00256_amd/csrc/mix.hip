// Shift-invariant gossip rounds for gfx950 (see ceca_mix_rounds in ceca.h): the comparison
// topologies of Table 1 -- ring, static exponential, one-peer exponential -- as circulant mixing of x.
#include <hip/hip_runtime.h>

#include "ceca.h"
#include "device_util.h"
#include "launch.h"

namespace ceca {

__device__ __forceinline__ float fma_each(float w, float z, float t) { return __builtin_fmaf(w, z, t); }
__device__ __forceinline__ vf4 fma_each(float w, vf4 z, vf4 t) {
  vf4 o;
  o.x = __builtin_fmaf(w, z.x, t.x); o.y = __builtin_fmaf(w, z.y, t.y);
  o.z = __builtin_fmaf(w, z.z, t.z); o.w = __builtin_fmaf(w, z.w, t.w);
  return o;
}

// Wavefronts per SIMD the kernel is compiled for: workgroups wider than 256 threads must fit 128
// registers per thread (one 1024-thread workgroup or two 512-thread ones per compute unit).
template <int THREADS>
constexpr int mix_waves() { return THREADS > 256 ? 4 : 1; }

// Same tiling as the fused CECA rounds: a workgroup keeps a column tile of every agent's x in
// registers (RT rows per thread) and publishes it in LDS once per round, where each row picks up its
// peers.  One read and one write of x for any number of rounds.
// SCALAR: weights in scalar instead of vector registers, see launch_mix.
template <int VEC, int RT, int THREADS, bool SCALAR>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(mix_waves<THREADS>())))
void mix_rounds_kernel(const MixArgs M) {
#pragma clang fp contract(off)
  using V = typename VecOf<VEC>::T;
  extern __shared__ float lds_x[];                 // [n][lanes] groups of VEC floats
  const int lanes = THREADS / M.row_lanes;
  const int tid = threadIdx.x;
  const int cg = tid % lanes;
  const int rg = tid / lanes;
  const int64_t tile = tile_of_block(M.mem.xcd_runs);
  if (tile * lanes >= M.ngroups) return;           // past the last tile (the grid is rounded up to whole runs)
  const int64_t g = tile * lanes + cg;
  const bool on = g < M.ngroups;
  const int64_t col = (on ? g : 0) * VEC;          // lanes past the last column shadow column group 0

  V x[RT];                                         // rows past the last agent shadow it
  const int64_t from = col - columns_back(M, col);
  load_rows<V, RT>(x, M.xin + from, M.ld, rg, M.row_lanes, M.n - 1, M.mem.cached_loads);
  if (M.mem.short_cols) {
    const int back = (int)(col - from);
#pragma unroll
    for (int k = 0; k < RT; ++k) x[k] = own_columns(x[k], back);
  }
  V* xs = reinterpret_cast<V*>(lds_x);
  // Row i, column group c sits in LDS slot i * lanes + c, so my row k is slot tid + k * THREADS
  // (row_lanes * lanes = THREADS).  rows_per_thread is the least that covers n, so only my last row can
  // lie past the last agent: it then holds what agent n - 1 does and is never published.
  constexpr int L = RT - 1;
  const bool last_mine = rg + L * M.row_lanes < M.n;
  const int wrap = in_vgpr(M.n * lanes * (int)sizeof(V));
  const uint32_t slot = lds_address(lds_x) + tid * sizeof(V), end = lds_address(lds_x) + wrap - sizeof(V);
  int spec = M.k0 % M.period;
  for (int t = 0; t < M.rounds; ++t) {
    const int j0 = M.start[spec], j1 = M.start[spec + 1];
    const float ws = SCALAR ? M.w_self[spec] : in_vgpr(M.w_self[spec]);
    if (j1 > j0) {                                  // a round without peers is the identity
#pragma unroll
      for (int k = 0; k < L; ++k) xs[tid + k * THREADS] = x[k];
      if (last_mine) xs[tid + L * THREADS] = x[L];
      __syncthreads();
      // peer by peer, all of the thread's rows at once: the RT LDS reads of a peer are independent and
      // issue back to back (row by row they would each wait for the one before).  Per row the order of
      // operations is t = w_self x, then t = fma(w_j, z_j, t) peer after peer -- with one peer that of the
      // CECA combine -- so the new x grows in the registers of the old one.
#pragma unroll
      for (int k = 0; k < RT; ++k) x[k] = ws * x[k];
      for (int j = j0; j < j1; ++j) {
        // The peer of row rg + k * row_lanes is `shift` rows back on the circle: from the near address while that is
        // inside the tile, from the far end otherwise.  One comparison and one select per row, with the rows'
        // distances constants of the load instructions: an addition and a wrap took four instructions and, with
        // their slower forms (a scalar operand, a minimum), more than the row's multiply-adds.
        const int shift = M.shift[j];
        const int past = shift - rg;               // rows k with k * row_lanes < past start from the far end
        uint32_t near = slot - shift * (lanes * (uint32_t)sizeof(V)), far = near + wrap;
        asm volatile("" : "+v"(near), "+v"(far));  // two addresses to select from, not one and a distance to add
        const float w = SCALAR ? M.w[j] : in_vgpr(M.w[j]);
        V z[RT];
#pragma unroll
        for (int k = 0; k < RT; ++k) {
          uint32_t q = k * M.row_lanes < past ? far : near;
          if (k == L) q = min(q + L * THREADS * (uint32_t)sizeof(V), end) - L * THREADS * (uint32_t)sizeof(V);   // a shadow row stays inside the tile
          z[k] = lds_load<V>(q + k * THREADS * (uint32_t)sizeof(V));
        }
        __builtin_amdgcn_sched_barrier(0);         // every read is issued before the first value is used
#pragma unroll
        for (int k = 0; k < RT; ++k) x[k] = fma_each(w, z[k], x[k]);
      }
      __syncthreads();
    }
    if (++spec == M.period) spec = 0;
  }
  if (!on) return;
  // the row addresses are worked out here, after the rounds: nothing of them occupies registers meanwhile
  int rg_out = rg;
  int64_t out = col;
  asm volatile("" : "+v"(rg_out), "+v"(out));
  store_rows<V, RT>(x, M.xout + out, M.ld, rg_out, M.row_lanes, M.n - 1, columns_back(M, out), M.mem.cached_stores);
}


// Vector registers for the weights are the rule (static exponential, 2^26 elements, vector against scalar: n = 258
// 304 us against 355, n = 600 336 against 385, n = 1026 427 against 539).  512-thread tiles with 32-byte rows and 6 or 7 rows
// per thread, which many peers per round take from 1281 agents on, are the exception up to 1664 agents, over five pitches:
// n = 1300 380 to 660 against 348 to 571, n = 1500 402 to 529 against 359 to 481, n = 1660 464 to 566 against 425 to 521
// (1281: 327 to 522 against 344 to 548); beyond, vector registers win again (n = 1700 465 to 555 against 496 to 604).
template <int VEC, int RT, int THREADS>
static hipError_t launch_mix(const MixArgs& mm, unsigned blocks, size_t lds, hipStream_t st) {
  auto fn = &mix_rounds_kernel<VEC, RT, THREADS, false>;
  if constexpr (VEC == 4 && THREADS == 512 && (RT == 6 || RT == 7))
    if (THREADS / mm.row_lanes * 16 < 64 && mm.n <= 13 * 128) fn = &mix_rounds_kernel<VEC, RT, THREADS, true>;
  if (lds > 64 * 1024) {
    // more than 64 KB of LDS per workgroup has to be asked for
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  fn<<<dim3(blocks), dim3(THREADS), lds, st>>>(mm);
  return hipGetLastError();
}

// 256-thread workgroups: up to 32 rows per thread
template <int VEC>
static hipError_t launch_mix_256(const MixArgs& mm, unsigned blocks, size_t lds, hipStream_t st) {
  switch (mm.rows_per_thread) {
#define CECA_RT(RT) case RT: return launch_mix<VEC, RT, 256>(mm, blocks, lds, st)
    CECA_RT(1); CECA_RT(2); CECA_RT(3); CECA_RT(4); CECA_RT(5); CECA_RT(6); CECA_RT(7); CECA_RT(8);
    CECA_RT(9); CECA_RT(10); CECA_RT(11); CECA_RT(12); CECA_RT(13); CECA_RT(14); CECA_RT(15); CECA_RT(16);
    CECA_RT(17); CECA_RT(18); CECA_RT(19); CECA_RT(20); CECA_RT(21); CECA_RT(22); CECA_RT(23); CECA_RT(24);
    CECA_RT(25); CECA_RT(26); CECA_RT(27); CECA_RT(28); CECA_RT(29); CECA_RT(30); CECA_RT(31); CECA_RT(32);
#undef CECA_RT
  }
  return hipErrorInvalidValue;
}

// wider workgroups (16-byte groups only): up to kMixWideRows rows per thread fit their 128 registers
template <int THREADS>
static hipError_t launch_mix_wide(const MixArgs& mm, unsigned blocks, size_t lds, hipStream_t st) {
  switch (mm.rows_per_thread) {
#define CECA_RT(RT) case RT: return launch_mix<4, RT, THREADS>(mm, blocks, lds, st)
    CECA_RT(1); CECA_RT(2); CECA_RT(3); CECA_RT(4); CECA_RT(5); CECA_RT(6); CECA_RT(7); CECA_RT(8);
    CECA_RT(9); CECA_RT(10); CECA_RT(11); CECA_RT(12); CECA_RT(13); CECA_RT(14); CECA_RT(15); CECA_RT(16);
#undef CECA_RT
  }
  return hipErrorInvalidValue;
}

hipError_t launch_mix_rounds(const MixArgs& m, bool vec4, hipStream_t st) {
  if (m.ngroups <= 0) return hipSuccess;
  const int threads = m.threads > 0 ? m.threads : kBlock;
  if (threads != 256 && threads != 512 && threads != 1024) return hipErrorInvalidValue;
  if (!vec4 && threads != 256) return hipErrorInvalidValue;          // scalar columns: 256-thread tiles only
  if (m.row_lanes < 1 || m.row_lanes > threads || (m.row_lanes & (m.row_lanes - 1)) != 0) return hipErrorInvalidValue;
  // the kernel relies on rows_per_thread being the least that covers n (only a thread's last row can
  // lie past the last agent)
  if (m.rows_per_thread < 1 || m.rows_per_thread > 32 ||
      (int64_t)m.rows_per_thread * m.row_lanes < m.n || (int64_t)(m.rows_per_thread - 1) * m.row_lanes >= m.n)
    return hipErrorInvalidValue;
  const int lanes = threads / m.row_lanes;
  int64_t blocks = (m.ngroups + lanes - 1) / lanes;
  if (blocks < 1 || blocks >= (1LL << 24)) return hipErrorInvalidConfiguration;
  MixArgs mm = m;
  tile_memory(&mm.mem, lanes * (vec4 ? 16 : 4), m.xin, m.xout, m.ld, &blocks);
  const size_t lds = (size_t)m.n * lanes * (vec4 ? 16 : 4);
  if (lds > kMultiMaxLds) return hipErrorInvalidValue;
  if (!vec4) return launch_mix_256<1>(mm, (unsigned)blocks, lds, st);
  if (threads == 256) return launch_mix_256<4>(mm, (unsigned)blocks, lds, st);
  if (threads == 512) return launch_mix_wide<512>(mm, (unsigned)blocks, lds, st);
  return launch_mix_wide<1024>(mm, (unsigned)blocks, lds, st);
}

}  // namespace ceca
