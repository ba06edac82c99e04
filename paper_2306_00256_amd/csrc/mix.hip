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
template <int VEC, int RT, int THREADS, bool WHOLE>
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
  const auto mem = tile_of<WHOLE>(M);
  const int64_t from = col - (WHOLE ? 0 : columns_back(M, col));
  load_rows<V, RT>(x, M.xin + from, M.ld, rg, M.row_lanes, M.n - 1, mem.cached_loads);
  if (mem.short_cols) {
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
    const float ws = in_vgpr(M.w_self[spec]);
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
        const float w = in_vgpr(M.w[j]);
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
  store_rows<V, RT>(x, M.xout + out, M.ld, rg_out, M.row_lanes, M.n - 1, WHOLE ? 0 : columns_back(M, out), mem.cached_stores);
}

// x <- w_self x + the terms of the round's first RUN peers, which are 1, 2, 4, 8 rows back: among the block's own rows or the
// REACH rows in front of it.  From the last row down, a row's own peers still hold their old values when its turn comes.
constexpr int lead_reach(int run) { return run > 0 ? 1 << (run - 1) : 0; }
template <int RUN, int RT>
__device__ __forceinline__ void mix_lead(vf4 (&x)[RT], uint32_t front, uint32_t pitch, float ws, const float* w) {
#pragma clang fp contract(off)
  constexpr int REACH = lead_reach(RUN);
  if constexpr (REACH < RT) {
    float wj[RUN];
#pragma unroll
    for (int j = 0; j < RUN; ++j) wj[j] = in_vgpr(w[j]);
    vf4 z[REACH];
#pragma unroll
    for (int k = 0; k < REACH; ++k) z[k] = lds_load<vf4>(front + k * pitch);
#pragma unroll
    for (int k = RT - 1; k >= 0; --k) {
      x[k] = ws * x[k];
#pragma unroll
      for (int j = 0; j < RUN; ++j) x[k] = fma_each(wj[j], k < 1 << j ? z[k - (1 << j) + REACH] : x[k - (1 << j)], x[k]);
      __builtin_amdgcn_sched_barrier(0);         // row by row: 7 rows then fit three 512-thread workgroups (80 registers, not 82)
    }
  }
}

// Wavefronts per SIMD: two 1024-thread workgroups of up to 5 rows are resident.
template <int THREADS, int RT>
constexpr int block_waves() { return THREADS == 1024 && RT <= 5 ? 8 : mix_waves<THREADS>(); }

// The same rounds with RT consecutive rows per thread: agents rg * RT and on.  A peer's rows are then consecutive as well, so
// one address per peer serves the whole block, its rows' distances being constants of the load instructions (rows row_lanes
// apart take a comparison and a select each), and the peers 1, 2, 4, 8 rows back are mostly the block's own rows, which are in
// registers: of static exponential's 99 LDS reads per thread and round at n = 1026 this leaves 71.  The tile is followed by
// copies of its first RT - 1 rows, so that no block of peers has a wrap inside.
// What bounds it: vector units (4.2 cycles per wavefront instruction and SIMD, of which 87 % are the rows' products) and
// LDS (busy 64 % of the time) together, n = 1026.
// Bank conflicts: lanes of a wavefront that differ in the row are RT rows apart, so rows of the tile that are less than all
// banks wide (LANES < 16) need an odd RT.  Same order of operations per row as above, same bits.
// Static exponential, 2^27 elements at pitches that are no power of two, rows row_lanes apart -> blocks: n = 100 401 -> 355 us,
// n = 130 496 -> 404, n = 258 611 -> 499, n = 500 686 -> 552, n = 800 684 -> 618, n = 1026 852 -> 715, n = 1400 967 -> 759, n = 2050 1010 -> 858.
// (At powers of two: n = 130, d = 2^20 520 -> 440, n = 1026, d = 2^17 901 -> 798.)  <1024, 4, 5> spills one register, for two resident
// workgroups.
template <int THREADS, int LANES, int RT>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(block_waves<THREADS, RT>())))
void mix_blocks_kernel(const MixArgs M) {
#pragma clang fp contract(off)
  extern __shared__ float lds_x[];                 // [n + RT - 1][LANES] groups of 4 floats
  constexpr uint32_t PITCH = LANES * sizeof(vf4);
  const int tid = threadIdx.x;
  const int cg = tid % LANES;
  const int rg = tid / LANES;
  const int64_t tile = tile_of_block(M.mem.xcd_runs);
  if (tile * LANES >= M.ngroups) return;           // past the last tile (the grid is rounded up to whole runs)
  const int64_t g = tile * LANES + cg;
  const bool on = g < M.ngroups;
  const int64_t col = (on ? g : 0) * 4;            // lanes past the last column shadow column group 0

  // Rows past agent n - 1 hold what the agents from 0 on do, and every block past it starts at agent n - 1.  Such rows are
  // worked out and published like any other, with the bits of the rows they stand for, so nothing below is conditional: the
  // first block past the last agent (the launcher sees to it that there is one) publishes the copies behind the tile.
  // Wavefronts that hold later blocks only just take part in the barriers.
  const int row0 = min(rg * RT, M.n - 1);
  const bool idle = (__builtin_amdgcn_readfirstlane(rg) - 1) * RT >= M.n;
  vf4 x[RT];
  const int64_t from = col - columns_back(M, col);
  if (!idle) {
    load_rows<vf4, RT, true>(x, M.xin + from, M.ld, row0, 1, M.n - 1, M.mem.cached_loads);
    if (M.mem.short_cols) {
      const int back = (int)(col - from);
#pragma unroll
      for (int k = 0; k < RT; ++k) x[k] = own_columns(x[k], back);
    }
  }
  const uint32_t wrap = M.n * PITCH;
  const uint32_t slot = lds_address(lds_x) + row0 * PITCH + cg * (uint32_t)sizeof(vf4);
  int spec = M.k0 % M.period;
  for (int t = 0; t < M.rounds; ++t) {
    int j = M.start[spec];
    const int j1 = M.start[spec + 1], run = M.lead[spec];
    if (j1 > j) {                                   // a round without peers is the identity
      // the first of the peers that are read from the tile, requested ahead like the ones after it
      j += run;
      int shift = M.shift[min(j, kMixMaxPeers - 1)];
      float weight = M.w[min(j, kMixMaxPeers - 1)];
      const float ws = in_vgpr(M.w_self[spec]);
      if (!idle) {
#pragma unroll
        for (int k = 0; k < RT; ++k) lds_store(slot + k * PITCH, x[k]);
      }
      __syncthreads();
      if (!idle) {
        // the block `shift` rows back on the circle
        auto back = [&](int shift) { return slot - shift * PITCH + (row0 < shift ? wrap : 0u); };
        switch (run) {
#define CECA_LEAD(RUN) case RUN: mix_lead<RUN, RT>(x, back(lead_reach(RUN)), PITCH, ws, M.w + M.start[spec]); break
          CECA_LEAD(1); CECA_LEAD(2); CECA_LEAD(3); CECA_LEAD(4);
#undef CECA_LEAD
          default:
#pragma unroll
            for (int k = 0; k < RT; ++k) x[k] = ws * x[k];
        }
        for (; j < j1; ++j) {
          const uint32_t q = back(shift);
          const float w = in_vgpr(weight);
          shift = M.shift[min(j + 1, kMixMaxPeers - 1)];
          weight = M.w[min(j + 1, kMixMaxPeers - 1)];
          // every read of a batch is issued before its first value is used; two batches where registers are short
          constexpr int KB = RT > 9 ? (RT + 1) / 2 : RT;
#pragma unroll
          for (int k0 = 0; k0 < RT; k0 += KB) {
            vf4 z[KB];
#pragma unroll
            for (int k = k0; k < k0 + KB && k < RT; ++k) z[k - k0] = lds_load<vf4>(q + k * PITCH);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = k0; k < k0 + KB && k < RT; ++k) x[k] = fma_each(w, z[k - k0], x[k]);
            if (KB < RT) __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      __syncthreads();
    }
    if (++spec == M.period) spec = 0;
  }
  if (!on || rg * RT >= M.n) return;
  // the row addresses are worked out here, after the rounds: nothing of them occupies registers meanwhile
  int row_out = row0;
  int64_t out = col;
  asm volatile("" : "+v"(row_out), "+v"(out));
  store_rows<vf4, RT>(x, M.xout + out, M.ld, row_out, 1, M.n - 1, columns_back(M, out), M.mem.cached_stores);
}


// Ring rounds (peers 1 row back and 1 ahead, in every round): a thread holds RT consecutive rows or one less, and of a block only
// its first and last row are anyone else's business.  They alone go through LDS, one slot per thread and two buffers in turn, so a
// round has one barrier and the tile's width is not bound by LDS: its rows are 256 bytes up to 448 agents, 128 up to 960 and 64 beyond,
// where a tile that keeps every row in LDS has 64 from 513 agents on.  A row's new value replaces it from the last one down, with the old value of the row
// behind carried along.  Same order of operations per row as above, same bits.
// What bounds it: memory (n = 1026 241 us where the loads and stores alone take 243 in the general form's tile).  Ring, 2^27 elements at
// pitches that are no power of two, general form -> here: n = 130 234 -> 193 us, n = 400 256 -> 217, n = 800 284 -> 217, n = 1026 333 ->
// 241, n = 1500 550 -> 251, n = 3000 614 -> 356.  (Powers of two: n = 130, d = 2^20 256 -> 212, n = 1026, d = 2^17 407 -> 309.)  Blocks of
// 15 rows spill 2 registers, those of 16 rows in 1024-thread workgroups (3841 agents on) 10.
template <int THREADS, int LANES, int RT, bool WHOLE>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(mix_waves<THREADS>())))
void mix_ring_kernel(const MixArgs M) {
#pragma clang fp contract(off)
  constexpr int ROW_LANES = THREADS / LANES;
  __shared__ vf4 first_row[2][THREADS], last_row[2][THREADS];
  const int tid = threadIdx.x;
  const int cg = tid % LANES;
  const int rg = tid / LANES;
  const int64_t tile = tile_of_block(M.mem.xcd_runs);
  if (tile * LANES >= M.ngroups) return;           // past the last tile (the grid is rounded up to whole runs)
  const int64_t g = tile * LANES + cg;
  const bool on = g < M.ngroups;
  const int64_t col = (on ? g : 0) * 4;            // lanes past the last column shadow column group 0

  const int whole = M.n - (RT - 1) * ROW_LANES;    // blocks of RT rows (1 to ROW_LANES), the others have one less
  const bool last_mine = rg < whole;
  const int agent = rg * (RT - 1) + min(rg, whole);
  const int last = agent + RT - 2 + last_mine;
  vf4 x[RT];                                       // the row that a shorter block lacks shadows its last one
  const auto mem = tile_of<WHOLE>(M);
  const int64_t from = col - (WHOLE ? 0 : columns_back(M, col));
  load_rows<vf4, RT>(x, M.xin + from, M.ld, agent, 1, last, mem.cached_loads);
  if (mem.short_cols) {
    const int back = (int)(col - from);
#pragma unroll
    for (int k = 0; k < RT; ++k) x[k] = own_columns(x[k], back);
  }
  const int before = rg > 0 ? tid - LANES : tid + THREADS - LANES;
  const int behind = rg < ROW_LANES - 1 ? tid + LANES : cg;
  int spec = M.k0 % M.period;
  for (int t = 0; t < M.rounds; ++t) {
    const int j = M.start[spec];
    const float ws = in_vgpr(M.w_self[spec]), wb = in_vgpr(M.w[j]), wa = in_vgpr(M.w[j + 1]);
    first_row[t & 1][tid] = x[0];
    last_row[t & 1][tid] = last_mine ? x[RT - 1] : x[RT - 2];
    __syncthreads();                               // the buffer's readers of two rounds ago have passed the barrier of the last one
    const vf4 front = last_row[t & 1][before];
    vf4 next = first_row[t & 1][behind];
#pragma unroll
    for (int k = RT - 1; k >= 0; --k) {
      const vf4 was = x[k];
      vf4 v = ws * was;
      v = fma_each(wb, k > 0 ? x[k > 0 ? k - 1 : 0] : front, v);
      x[k] = fma_each(wa, next, v);
      next = k == RT - 1 && !last_mine ? next : was;
      if (RT > 8) __builtin_amdgcn_sched_barrier(0);       // row by row where registers are short
    }
    if (++spec == M.period) spec = 0;
  }
  if (!on) return;
  // the row addresses are worked out here, after the rounds: nothing of them occupies registers meanwhile
  int row_out = agent;
  int64_t out = col;
  asm volatile("" : "+v"(row_out), "+v"(out));
  store_rows<vf4, RT>(x, M.xout + out, M.ld, row_out, 1, last, WHOLE ? 0 : columns_back(M, out), mem.cached_stores);
}

template <int VEC, int RT, int THREADS>
static hipError_t launch_mix(const MixArgs& mm, unsigned blocks, size_t lds, hipStream_t st) {
  auto fn = &mix_rounds_kernel<VEC, RT, THREADS, false>;
  if constexpr (VEC == 4 && THREADS <= 512)
    if (mm.mem.whole()) fn = &mix_rounds_kernel<VEC, RT, THREADS, true>;
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

// Rows per thread of the form with blocks of consecutive rows for this tile, 0 where there is none: enough that at least one
// block lies past the last agent; the next odd number where rows of the tile are narrower than 256 bytes (bank conflicts, see the
// kernel).  For many peers per round from 97 agents on: wider rows of the tile, below that, lose (n = 64 296 us against 322,
// n = 80 376 against 379), and so does one peer, which hides behind the memory traffic (one-peer exponential, n = 1026 277
// against 321, n = 500 236 against 274).  512-thread tiles of 64-byte rows from 672 agents on only: with 635, 71 % of the blocks
// are in use, 647 us against 689, with 513 to 634 no difference, n = 700 708 against 672.
static int block_rows(const MixArgs& m, int threads, int lanes) {
  int most = 0;
  for (int q = 0; q < m.period; ++q) most = most > m.start[q + 1] - m.start[q] ? most : m.start[q + 1] - m.start[q];
  if (most < 4 || lanes > 16) return 0;
  int rows = m.n / (threads / lanes - 1) + 1;
  if (lanes < 16) rows |= 1;
  switch (threads) {
    case 256: return lanes == 16 ? (rows >= 7 && rows <= 13 ? rows : 0) : (lanes == 8 && rows >= 7 && rows <= 17 ? rows : 0);
    case 512: return lanes == 4 ? (m.n >= 672 && rows <= 9 ? rows : 0) : (lanes == 2 && rows >= 7 && rows <= 9 ? rows : 0);
    case 1024: return lanes == 4 && rows == 5 ? rows : 0;
  }
  return 0;
}

template <int THREADS, int LANES, int RT>
static hipError_t launch_blocks(const MixArgs& mm, unsigned blocks, hipStream_t st) {
  const auto fn = &mix_blocks_kernel<THREADS, LANES, RT>;
  const size_t lds = (size_t)(mm.n + RT - 1) * LANES * 16;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  fn<<<dim3(blocks), dim3(THREADS), lds, st>>>(mm);
  return hipGetLastError();
}
static hipError_t launch_mix_blocks(const MixArgs& mm, int lanes, int rows, unsigned blocks, hipStream_t st) {
  switch (mm.threads << 16 | lanes << 8 | rows) {
#define CECA_RT(T, L, RT) case T << 16 | L << 8 | RT: return launch_blocks<T, L, RT>(mm, blocks, st)
    CECA_RT(256, 16, 7); CECA_RT(256, 16, 8); CECA_RT(256, 16, 9); CECA_RT(256, 16, 10); CECA_RT(256, 16, 11); CECA_RT(256, 16, 12); CECA_RT(256, 16, 13);
    CECA_RT(256, 8, 7); CECA_RT(256, 8, 9); CECA_RT(256, 8, 11); CECA_RT(256, 8, 13); CECA_RT(256, 8, 15); CECA_RT(256, 8, 17);
    CECA_RT(512, 4, 7); CECA_RT(512, 4, 9);
    CECA_RT(512, 2, 7); CECA_RT(512, 2, 9);
    CECA_RT(1024, 4, 5);
#undef CECA_RT
  }
  return hipErrorInvalidValue;
}

// How many of the round's first peers are 1, 2, 4, 8 rows back in this order and less than a block of `rows` rows.
static int lead_of(const MixArgs& m, int spec, int rows) {
  const int32_t* s = m.shift + m.start[spec];
  const int peers = m.start[spec + 1] - m.start[spec];
  int run = 0;
  while (run < peers && run < 4 && s[run] == 1 << run && 1 << run < rows) ++run;
  return run;
}

// Threads and column groups per row of the ring kernel's tile; false where the rounds are no ring rounds, the tile is prescribed,
// or there are so few agents that the general form's rows are as wide.  Rows of the tile as wide as registers allow (about 15 rows
// per thread in 512-thread workgroups: with 17, n = 1026 410 us against 241 at 9 rows of half the width), 2^27 elements at
// three pitches, the narrower or the smaller of the two against the choice: n = 130 212 / 198 / 257 us (128-byte rows) against 193 /
// 194 / 235; n = 300 223 / 203 / 261 (256 threads) against 211 / 210 / 234; n = 917 268 / 264 / 331 (64-byte rows) against 247 / 221 /
// 271; n = 1500 244 / 235 / 296 (1024 threads) against 251 / 235 / 303; n = 2050 523 / 535 / 581 (512 threads) against 364 / 361 / 424.
static bool ring_tile(const MixArgs& m, int* threads, int* lanes) {
  if (m.n <= 64 || g_tuning.rows || g_tuning.tile_threads) return false;
  for (int q = 0; q < m.period; ++q)
    if (m.start[q + 1] - m.start[q] != 2 || m.shift[m.start[q]] != 1 || m.shift[m.start[q] + 1] != m.n - 1) return false;
  *threads = m.n <= 272 ? 256 : m.n <= 1792 ? 512 : 1024;
  *lanes = m.n <= 448 ? 16 : m.n <= 960 ? 8 : 4;
  return true;
}

static hipError_t launch_mix_ring(const MixArgs& mm, int threads, int lanes, unsigned blocks, hipStream_t st) {
  const int row_lanes = threads / lanes, rows = (mm.n + row_lanes - 1) / row_lanes;
  switch (threads << 16 | lanes << 8 | rows) {
#define CECA_RT(T, L, RT) case T << 16 | L << 8 | RT: (mm.mem.whole() ? &mix_ring_kernel<T, L, RT, true> : &mix_ring_kernel<T, L, RT, false>)<<<dim3(blocks), dim3(T), 0, st>>>(mm); return hipGetLastError()
#define CECA_RTS(T, L) CECA_RT(T, L, 8); CECA_RT(T, L, 9); CECA_RT(T, L, 10); CECA_RT(T, L, 11); CECA_RT(T, L, 12); CECA_RT(T, L, 13); CECA_RT(T, L, 14)
    CECA_RT(256, 16, 5); CECA_RT(256, 16, 6); CECA_RT(256, 16, 7); CECA_RTS(256, 16); CECA_RT(256, 16, 15); CECA_RT(256, 16, 16); CECA_RT(256, 16, 17);
    CECA_RTS(512, 16); CECA_RTS(512, 8); CECA_RT(512, 8, 15); CECA_RTS(512, 4); CECA_RTS(1024, 4); CECA_RT(1024, 4, 15); CECA_RT(1024, 4, 16);
#undef CECA_RTS
#undef CECA_RT
  }
  return hipErrorInvalidValue;
}

bool mix_in_blocks(const MixArgs& m) {
  int threads, lanes;
  return ring_tile(m, &threads, &lanes) || block_rows(m, m.threads, m.threads / m.row_lanes) > 0;
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
  int lanes = threads / m.row_lanes, ring_threads = 0;
  const bool ring = vec4 && ring_tile(m, &ring_threads, &lanes);
  int64_t blocks = (m.ngroups + lanes - 1) / lanes;
  if (blocks < 1 || blocks >= (1LL << 24)) return hipErrorInvalidConfiguration;
  MixArgs mm = m;
  tile_memory(&mm.mem, lanes * (vec4 ? 16 : 4), m.xin, m.xout, m.ld, m.n, &blocks, nullptr, 0, /*narrow_streamed=*/!ring);
  if (ring) return launch_mix_ring(mm, ring_threads, lanes, (unsigned)blocks, st);
  const size_t lds = (size_t)m.n * lanes * (vec4 ? 16 : 4);
  if (lds > kMultiMaxLds) return hipErrorInvalidValue;
  mm.threads = threads;
  const int rows = vec4 ? block_rows(m, threads, lanes) : 0;
  if (rows) {
    for (int q = 0; q < m.period; ++q) mm.lead[q] = lead_of(m, q, rows);
    return launch_mix_blocks(mm, lanes, rows, (unsigned)blocks, st);
  }
  if (!vec4) return launch_mix_256<1>(mm, (unsigned)blocks, lds, st);
  if (threads == 256) return launch_mix_256<4>(mm, (unsigned)blocks, lds, st);
  if (threads == 512) return launch_mix_wide<512>(mm, (unsigned)blocks, lds, st);
  return launch_mix_wide<1024>(mm, (unsigned)blocks, lds, st);
}

}  // namespace ceca
