// Minibatch gradients of the GEMV-shaped losses for gfx950: margins a_ij . z_i, then e_i and the message.
#include <hip/hip_runtime.h>

#include "ceca.h"
#include "device_util.h"
#include "gemv_util.h"
#include "launch.h"

namespace ceca {

// Minibatch row numbers are the same for every lane: keep them in scalar registers so that row
// addresses are scalar and all row loads can be issued back to back.
__device__ __forceinline__ int32_t uniform_i32(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
// Sampled row numbers are forced into [0, N) wherever they are used: a bad index must not become a
// wild read.

// Sampled rows are not moved where a row's last group is short (own_columns): the lane takes the row's last four columns
// as they lie, its z is moved to meet them for the dot products (zeros for its neighbour's columns), and its gradient is
// moved to its own columns once it is summed.  Both are skipped by wavefronts without such a lane.
// Zero times an infinite feature is NaN, and a NaN margin makes the whole message NaN where an infinite one loses that feature's
// column alone.  So where the products of a wavefront have a NaN they are taken again with zeros for what is not the
// lane's own (own_of_row).  (Rows of whole groups keep one way to a NaN: lanes past the last column read the row's first group.)
template <bool ODD, typename V> __device__ __forceinline__ V z_for_rows(V z, int back) { return ODD && __any(back != 0) ? last_columns(z, back) : z; }
template <bool ODD, typename V> __device__ __forceinline__ V own_gradient(V e, int back) { return ODD && __any(back != 0) ? own_columns(e, back) : e; }
// partial[(agent * nchunks + chunk) * B + j] = sum over the chunk's columns of A[row_j][col] * z[agent][col].
// A workgroup takes one column chunk of kRowGroup sampled rows of one agent (grid: chunks x agents x row groups),
// so few agents still spread over many workgroups.
// FUSE: the workgroup first finishes the iteration before for its agent and columns -- x+, y+ from x, y,
// its own message and its peer's (Eqs. (8), (9), with the arithmetic of the combine kernel, operation
// for operation) -- and takes the margins at the new z.  Every row group of an (agent, chunk) pair
// computes the same x+, y+; the first one stores them, into a buffer other than the one they are read
// from (the row groups run at the same time).
template <int VEC, bool ODD, bool FUSE>
__global__ __launch_bounds__(kBlock) void margins_kernel(const GemvArgs G) {
  using V = typename VecOf<VEC>::T;
  __shared__ float red[kBlock / 64][kRowGroup];
  const int agent = blockIdx.y;
  const int chunk = blockIdx.x;
  const int j0 = blockIdx.z * kRowGroup;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

  // lanes past the last column read column 0 instead and carry z = 0: no branch surrounds a load
  const int64_t c = (int64_t)chunk * G.chunk_cols + (int64_t)threadIdx.x * VEC;
  const bool on = c < G.d;
  const int64_t col = on ? c : 0;
  const int back = short_back<ODD>(col, G.d);
  V zv;
  if (FUSE) {
#pragma clang fp contract(off)
    int p;
    if (G.p_port == 2) {
      p = agent - G.p_shift; if (p < 0) p += G.n;
    } else {
      p = (agent & 1) ? agent - G.p_shift : agent + G.p_shift;
      if (p < 0) p += G.n;
      if (p >= G.n) p -= G.n;
    }
    const int64_t off = (int64_t)agent * G.ld + col;
    const V x = ld_own<V>(G.px + off, back);
    const V y = G.p_read_y || G.p_exch_y ? ld_own<V>(G.py + off, back) : V(0.0f);
    const V v = ld_plain<V>(G.pv + (int64_t)agent * G.ldv + col);
    const V msg = ld_plain<V>(G.pv + (int64_t)p * G.ldv + col);
    const V dz = v - (G.p_exch_y ? y : x);          // -lr e of the iteration before
    const V xs = G.p_exch_y ? x + dz : v;
    const V ys = G.p_exch_y ? v : y + dz;
    const V xn = combine(G.pa, xs, G.pap, msg);
    const V yn = G.p_read_y ? combine(G.pb, ys, G.pbp, msg) : G.pbp * msg;
    if (on && blockIdx.z == 0) {
      const int64_t oo = (int64_t)agent * G.ldo + col;
      st_own<V>(G.ox + oo, xn, back);
      st_own<V>(G.oy + oo, yn, back);
    }
    zv = G.new_exch_y ? yn : xn;
  } else {
    zv = ld_own<V>(G.zin + (int64_t)agent * G.ld + col, back);
  }
  const V z = on ? z_for_rows<ODD>(zv, back) : V(0.0f);
  const int32_t* idx = G.batch_idx + (int64_t)agent * G.B;
  const float* Abase = G.A + (int64_t)agent * G.N * G.lda + col - back;
  // one vector load for the group's sample numbers (lane jj holds sample j0 + jj; samples past B repeat
  // the last), made scalar lane by lane: scalar loads would each wait for the one before
  const int32_t myidx = idx[min(j0 + min(lane, kRowGroup - 1), G.B - 1)];
  V a[kRowGroup];
#pragma unroll
  for (int jj = 0; jj < kRowGroup; ++jj) {
    const int32_t rj = min(max(__builtin_amdgcn_readlane(myidx, jj), 0), G.N - 1);
    a[jj] = ld_stream<V>(Abase + (int64_t)rj * G.lda);
  }
  float acc[kRowGroup];
#pragma unroll
  for (int jj = 0; jj < kRowGroup; ++jj) acc[jj] = dot_v(a[jj], z);
  if (ODD && some_nan(acc)) {
#pragma unroll
    for (int jj = 0; jj < kRowGroup; ++jj) acc[jj] = dot_v(own_of_row(a[jj], columns_left(c, G.d)), z);
  }
  int jj;
  bool owner;
  const float s = wave_sum_many<kRowGroup>(acc, lane, jj, owner);
  if (owner) red[wave][jj] = s;
  __syncthreads();
  if ((int)threadIdx.x < kRowGroup && j0 + (int)threadIdx.x < G.B) {
    float t = 0.0f;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) t += red[w][threadIdx.x];
    G.partial[((int64_t)agent * G.nchunks + chunk) * G.B + j0 + threadIdx.x] = t;
  }
}

// v_i = z_i - lr * e_i with e_i = sum_j coef_j a_ij; coef_j folds the loss derivative and the 1/B.
template <int VEC, bool ODD>
__global__ __launch_bounds__(kBlock) void halfstep_kernel(const GemvArgs G) {
  using V = typename VecOf<VEC>::T;
  __shared__ float coef[64 + kRowGroup];
  __shared__ int32_t rowid[64 + kRowGroup];
  const int agent = blockIdx.y;
  if ((int)threadIdx.x < 64 + kRowGroup) {
    const int j = min((int)threadIdx.x, G.B - 1);
    float m = 0.0f;
    for (int ch = 0; ch < G.nchunks; ++ch) m += G.partial[((int64_t)agent * G.nchunks + ch) * G.B + j];
    const int32_t row = min(max(G.batch_idx[(int64_t)agent * G.B + j], 0), G.N - 1);
    const float t = G.t[(int64_t)agent * G.N + row];
    // entries past B repeat the last row with coefficient 0, so the row loop needs no bounds test
    coef[threadIdx.x] = ((int)threadIdx.x < G.B) ? loss_coef(G.kind, m, t, G.scale) : 0.0f;
    rowid[threadIdx.x] = row;
  }
  __syncthreads();
  const int64_t col = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * VEC;
  if (col >= G.d) return;
  const int back = short_back<ODD>(col, G.d);
  V e = V(0.0f);
  const float* base = G.A + (int64_t)agent * G.N * G.lda + col - back;
  for (int j0 = 0; j0 < G.B; j0 += kRowGroup) {
    V r[kRowGroup];
#pragma unroll
    for (int jj = 0; jj < kRowGroup; ++jj) r[jj] = ld_stream<V>(base + (int64_t)uniform_i32(rowid[j0 + jj]) * G.lda);
#pragma unroll
    for (int jj = 0; jj < kRowGroup; ++jj) e += coef[j0 + jj] * r[jj];
  }
  e = own_gradient<ODD>(e, back);
  if (G.noise_std != 0.0f) e = add_noise<V>(e, G.noise_std, col, noise_keys(G.seed, G.k, (uint32_t)agent));
  const V z = ld_own<V>(G.zin + (int64_t)agent * G.ld + col, back);
  *reinterpret_cast<V*>(G.v + (int64_t)agent * G.ldv + col) = z - G.lr * e;     // (message rows have room for whole groups)
}

// One pass over the minibatch rows: a workgroup owns an agent, keeps its B sampled rows of A in
// registers (B x G 16-byte groups per thread), reduces the B margins across the workgroup, and forms
// v = z - lr * e from the same registers, so A is read from memory once per iteration.
template <int THREADS, int BMAX, int G, bool ODD>
__global__ __launch_bounds__(THREADS) void grad_onepass_kernel(const GemvArgs P) {
  constexpr int WAVES = THREADS / 64;
  __shared__ float red[2][WAVES][BMAX];   // alternating between a workgroup's agents: one barrier per agent
  static_assert(BMAX <= 64, "one lane per sampled row");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // lanes past the last column read column 0 instead and carry z = 0: no branch surrounds a load
  int64_t col[G];
  bool on[G];
  int back[G];
#pragma unroll
  for (int u = 0; u < G; ++u) {
    const int64_t c = ((int64_t)u * THREADS + threadIdx.x) * 4;
    on[u] = c < P.d;
    col[u] = on[u] ? c : 0;
    back[u] = short_back<ODD>(col[u], P.d);
  }
  // A workgroup takes agents blockIdx.x, blockIdx.x + gridDim.x, ...  The next agent's batch numbers
  // and z are requested while the current agent is being worked on, so only the first agent of a
  // workgroup waits for them before its rows can be requested.
  // One vector load brings a whole batch into a wavefront (lane j holds sample j; samples past B repeat
  // the last); the row numbers then become scalars lane by lane: B scalar loads would each wait for
  // the one before, because scalar loads return out of order.
  int agent = blockIdx.x;
  int32_t idx_next = P.batch_idx[(int64_t)agent * P.B + min(lane, P.B - 1)];
  vf4 z_next[G];
#pragma unroll
  for (int u = 0; u < G; ++u) z_next[u] = ld_plain<vf4>(P.zin + (int64_t)agent * P.ld + col[u] - back[u]);
  for (int turn = 0; agent < P.n; agent += gridDim.x, turn ^= 1) {
    const int32_t myidx = idx_next;
    vf4 z[G], zr[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {
      z[u] = on[u] ? own_gradient<ODD>(z_next[u], back[u]) : vf4(0.0f);
      zr[u] = z_for_rows<ODD>(z[u], back[u]);
    }
    const float* Abase = P.A + (int64_t)agent * P.N * P.lda;
    int32_t rowid[BMAX];
#pragma unroll
    for (int j = 0; j < BMAX; ++j) rowid[j] = min(max(__builtin_amdgcn_readlane(myidx, j), 0), P.N - 1);
    vf4 a[BMAX][G];
#pragma unroll
    for (int j = 0; j < BMAX; ++j) {
      const float* row = Abase + (int64_t)rowid[j] * P.lda;
#pragma unroll
      for (int u = 0; u < G; ++u) a[j][u] = ld_stream<vf4>(row + col[u] - back[u]);
    }
    // the target of "my" sampled row (lanes 0 .. BMAX-1 of every wavefront turn margins into
    // coefficients later) is requested here, behind the rows, so that nothing waits for it after the
    // barrier; the row number comes from the scalar row ids, so nothing has to arrive first
    int32_t rmine = rowid[0];
#pragma unroll
    for (int j = 1; j < BMAX; ++j) rmine = (lane == j) ? rowid[j] : rmine;
    const float tmine = P.t[(int64_t)agent * P.N + rmine];
    // what the next agent of this workgroup needs first (the last one re-reads its own: no branch)
    const int nxt = agent + (int)gridDim.x < P.n ? agent + (int)gridDim.x : agent;
    idx_next = P.batch_idx[(int64_t)nxt * P.B + min(lane, P.B - 1)];
#pragma unroll
    for (int u = 0; u < G; ++u) z_next[u] = ld_plain<vf4>(P.zin + (int64_t)nxt * P.ld + col[u] - back[u]);
    // every load above is issued before any arithmetic below: the scheduler must not trade loads in
    // flight for registers here (it split the rows into two dependent batches when left alone)
    __builtin_amdgcn_sched_barrier(0);
    float m[BMAX];
#pragma unroll
    for (int j = 0; j < BMAX; ++j) {
      m[j] = 0.0f;
#pragma unroll
      for (int u = 0; u < G; ++u) m[j] += dot_v(a[j][u], zr[u]);
    }
    if (ODD && some_nan(m)) {
#pragma unroll
      for (int j = 0; j < BMAX; ++j) {
        m[j] = 0.0f;
#pragma unroll
        for (int u = 0; u < G; ++u) m[j] += dot_v(own_of_row(a[j][u], columns_left(((int64_t)u * THREADS + threadIdx.x) * 4, P.d)), zr[u]);
      }
    }
    constexpr int CH = BMAX < 16 ? BMAX : 16;        // margins are summed across the wavefront 16 at a time
#pragma unroll
    for (int c0 = 0; c0 < BMAX; c0 += CH) {
      float part[CH];
#pragma unroll
      for (int k = 0; k < CH; ++k) part[k] = m[c0 + k];
      int jrow;
      bool owner;
      const float msum = wave_sum_many<CH>(part, lane, jrow, owner);
      if (owner) red[turn][wave][c0 + jrow] = msum;
    }
    __syncthreads();
    // every wavefront turns the margins into coefficients for itself (lane j: sample j, same summation
    // order everywhere), so no second barrier and no LDS round trip for the coefficients
    float cmine = 0.0f;
    {
      const int j = min(lane, BMAX - 1);
      float mj = 0.0f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) mj += red[turn][w][j];
      cmine = (lane < P.B) ? loss_coef(P.kind, mj, tmine, P.scale) : 0.0f;
    }
    float coef[BMAX];                                 // wavefront-uniform: scalar registers
#pragma unroll
    for (int j = 0; j < BMAX; ++j) coef[j] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, cmine), j));
#pragma unroll
    for (int u = 0; u < G; ++u) {
      vf4 e = vf4(0.0f);
#pragma unroll
      for (int j = 0; j < BMAX; ++j) e += coef[j] * a[j][u];
      e = own_gradient<ODD>(e, back[u]);
      if (P.noise_std != 0.0f) e = add_noise<vf4>(e, P.noise_std, col[u], noise_keys(P.seed, P.k, (uint32_t)agent));
      if (on[u]) *reinterpret_cast<vf4*>(P.v + (int64_t)agent * P.ldv + col[u]) = z[u] - P.lr * e;
    }
  }
}

// The same computation with the batch taken CH rows at a time: only CH rows of A are in registers at
// once, so two 1024-thread workgroups fit a compute unit and one computes while the other waits for
// its rows.  e accumulates over the samples in the same order as in the kernel above.
// (One column group per thread fits 64 registers, i.e. two 1024-thread workgroups per unit; wider rows
// take up to 128 registers and one such workgroup per unit, but still any batch size.)
// FUSE: the workgroup first finishes the iteration before for its agent -- x+, y+ from x, y, its own
// message and its peer's (Eqs. (8), (9), with the arithmetic of the combine kernel, operation for
// operation) -- stores them, and takes the gradient at the new z.  One launch per iteration instead
// of two, and the state rows (cache resident at these sizes) are touched once.
// FUSE = 2: the state between iterations is kept in half-step form -- rows xs = x - lr e, ys = y - lr e of
// the iteration before (the travelling one of the two IS that iteration's message, bit for bit) -- so the
// prologue reads its own two rows and one row of its peer, combines in registers without storing x+, y+,
// and the epilogue writes the new half-step rows to the other buffer: 20 bytes of state traffic per
// agent-parameter and iteration instead of 28, with the arithmetic of FUSE = 1 operation for operation.
// VEC = 1 is the same kernel on single columns (see minibatch_vec).  Of the instances only <4, 1024, 2, 4, 2, true> spills (9 registers:
// half-step runs on rows of more than 8192 columns that are no whole groups).
template <int VEC, int THREADS, int CH, int G, int FUSE, bool ODD>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(G == 1 ? 8 : 4, 8)))
void grad_chunked_kernel(const GemvArgs P) {
  using V = typename VecOf<VEC>::T;
  constexpr int WAVES = THREADS / 64;
  __shared__ float red[2][WAVES][CH];     // alternating between chunks: one barrier per chunk
  static_assert(CH <= 16, "one wavefront sum per chunk");
  const int agent = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t col[G];
  bool on[G];
  int back[G];
  V z[G], e[G];
  // FUSE = 2: the variable that does not travel this iteration, after the combine.  It is needed again only in
  // the epilogue and waits in LDS meanwhile (in registers it pushed three others out to scratch memory,
  // 8 MB of extra writes per iteration at n = 1023, d = 4096); a thread reads back what it wrote itself.
  __shared__ V other_s[FUSE == 2 ? THREADS * G : 1];
#pragma unroll
  for (int u = 0; u < G; ++u) {
    const int64_t c = ((int64_t)u * THREADS + threadIdx.x) * VEC;
    on[u] = c < P.d;
    col[u] = on[u] ? c : 0;
    back[u] = short_back<ODD>(col[u], P.d);
  }
  const float* Abase = P.A + (int64_t)agent * P.N * P.lda;
  // lane j holds sample j of the whole batch (B <= 64; samples past B repeat the last)
  const int32_t myidx = min(max(P.batch_idx[(int64_t)agent * P.B + min(lane, P.B - 1)], 0), P.N - 1);
  const float tmine = P.t[(int64_t)agent * P.N + myidx];
  V a[CH][G];
  // rows c0 .. c0 + CH - 1 of the batch into the register tile
  auto request_rows = [&](int c0) {
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const int32_t rj = __builtin_amdgcn_readlane(myidx, min(c0 + j, 63));
      const float* row = Abase + (int64_t)rj * P.lda;
#pragma unroll
      for (int u = 0; u < G; ++u) a[j][u] = ld_stream<V>(row + col[u] - back[u]);
    }
  };
  // without the prologue the first rows are requested before z; with it they follow it: the prologue
  // needs 24 registers of its own, and loads return in order anyway
  if (FUSE == 0) request_rows(0);
#pragma unroll
  for (int u = 0; u < G; ++u) {
    V zv;
    if (FUSE == 2) {
#pragma clang fp contract(off)
      const int64_t off = (int64_t)agent * P.ld + col[u];
      const V hx = ld_own<V>(P.px + off, back[u]);
      const V hy = ld_own<V>(P.py + off, back[u]);
      V xn = hx, yn = hy;                  // the call's first iteration starts from x, y themselves
      if (!P.p_first) {
        int p;
        if (P.p_port == 2) {
          p = agent - P.p_shift; if (p < 0) p += P.n;
        } else {
          p = (agent & 1) ? agent - P.p_shift : agent + P.p_shift;
          if (p < 0) p += P.n;
          if (p >= P.n) p -= P.n;
        }
        // the peer's message is the travelling row of its half-step state
        const V msg = ld_own<V>((P.p_exch_y ? P.py : P.px) + (int64_t)p * P.ld + col[u], back[u]);
        xn = combine(P.pa, hx, P.pap, msg);
        yn = P.p_read_y ? combine(P.pb, hy, P.pbp, msg) : P.pbp * msg;
      }
      zv = P.new_exch_y ? yn : xn;
      other_s[u * THREADS + threadIdx.x] = P.new_exch_y ? xn : yn;
    } else if (FUSE == 1) {
#pragma clang fp contract(off)
      int p;
      if (P.p_port == 2) {
        p = agent - P.p_shift; if (p < 0) p += P.n;
      } else {
        p = (agent & 1) ? agent - P.p_shift : agent + P.p_shift;
        if (p < 0) p += P.n;
        if (p >= P.n) p -= P.n;
      }
      const int64_t off = (int64_t)agent * P.ld + col[u];
      const V x = ld_own<V>(P.px + off, back[u]);
      const V y = P.p_read_y || P.p_exch_y ? ld_own<V>(P.py + off, back[u]) : V(0.0f);
      const V v = ld_plain<V>(P.pv + (int64_t)agent * P.ldv + col[u]);
      const V msg = ld_plain<V>(P.pv + (int64_t)p * P.ldv + col[u]);
      const V dz = v - (P.p_exch_y ? y : x);        // -lr e of the iteration before
      const V xs = P.p_exch_y ? x + dz : v;
      const V ys = P.p_exch_y ? v : y + dz;
      const V xn = combine(P.pa, xs, P.pap, msg);
      const V yn = P.p_read_y ? combine(P.pb, ys, P.pbp, msg) : P.pbp * msg;
      if (on[u]) {
        st_own<V>(P.ox + off, xn, back[u]);
        st_own<V>(P.oy + off, yn, back[u]);
      }
      zv = P.new_exch_y ? yn : xn;
    } else {
      zv = ld_own<V>(P.zin + (int64_t)agent * P.ld + col[u], back[u]);
    }
    z[u] = on[u] ? z_for_rows<ODD>(zv, back[u]) : V(0.0f);       // moved back below, with the gradient
    e[u] = V(0.0f);
  }
  if (FUSE != 0) request_rows(0);
  int turn = 0;
  for (int c0 = 0; c0 < P.B; c0 += CH, turn ^= 1) {
    float m[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      m[j] = 0.0f;
#pragma unroll
      for (int u = 0; u < G; ++u) m[j] += dot_v(a[j][u], z[u]);
    }
    if (ODD && some_nan(m)) {
#pragma unroll
      for (int j = 0; j < CH; ++j) {
        m[j] = 0.0f;
#pragma unroll
        for (int u = 0; u < G; ++u) m[j] += dot_v(own_of_row(a[j][u], columns_left(((int64_t)u * THREADS + threadIdx.x) * VEC, P.d)), z[u]);
      }
    }
    int jrow;
    bool owner;
    const float msum = wave_sum_many<CH>(m, lane, jrow, owner);
    if (owner) red[turn][wave][jrow] = msum;
    __syncthreads();
    // lane c0 + j of every wavefront turns margin j of this chunk into its coefficient
    const int jm = min(max(lane - c0, 0), CH - 1);
    float mj = 0.0f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) mj += red[turn][w][jm];
    const float cmine = (lane >= c0 && lane < P.B) ? loss_coef(P.kind, mj, tmine, P.scale) : 0.0f;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const float cj = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, cmine), min(c0 + j, 63)));
#pragma unroll
      for (int u = 0; u < G; ++u) e[u] += cj * a[j][u];
    }
    if (c0 + CH < P.B) request_rows(c0 + CH);       // same for every thread
  }
#pragma unroll
  for (int u = 0; u < G; ++u) {
    V ee = own_gradient<ODD>(e[u], back[u]);
    z[u] = own_gradient<ODD>(z[u], back[u]);
    if (P.noise_std != 0.0f) ee = add_noise<V>(ee, P.noise_std, col[u], noise_keys(P.seed, P.k, (uint32_t)agent));
    const V v = z[u] - P.lr * ee;
    if (FUSE == 2) {
      // half-step rows for the next iteration's combine: the travelling variable becomes the message itself,
      // the other moves by the same -lr e = v - z (the arithmetic of the combine kernel on stored messages)
      const V dz = v - z[u];
      const V moved = other_s[u * THREADS + threadIdx.x] + dz;
      if (on[u]) {
        const int64_t off = (int64_t)agent * P.ldo + col[u];
        st_own<V>(P.ox + off, P.new_exch_y ? moved : v, back[u]);
        st_own<V>(P.oy + off, P.new_exch_y ? v : moved, back[u]);
      }
    } else {
      if (on[u]) *reinterpret_cast<V*>(P.v + (int64_t)agent * P.ldv + col[u]) = v;
    }
  }
}

// Rows go in 16-byte groups whatever their base, pitch and length (own_columns), except those of up to 256 columns that
// are no whole groups: 64 or 256 threads hold those in single columns, with a quarter of the registers (window of n = 125, d = 199,
// B = 46: 2.8 us per iteration against 3.7 in groups; n = 360, d = 95, B = 25 7.6 against 8.2).  Longer ones gain: n = 60, d =
// 351, B = 17 8.0 -> 3.3 us per iteration, n = 600, d = 1547, B = 19 52 -> 29, n = 890, d = 1333, B = 53 133 -> 72, n = 313,
// d = 4510, B = 11 53 -> 26.
// Whole groups of up to 256 columns that do not lie on 16-byte boundaries take single columns too where a batch over 32 leaves
// groups few resident agents and no single-launch step, and up to 64 columns, which one wavefront holds: n = 391, d = 56, B = 40 6.9 us
// per iteration in groups against 2.8, n = 448, d = 12, B = 13 6.2 against 2.6, single steps of n = 12, d = 8, B = 56 10.0
// against 4.8; with 65 to 256 columns and B <= 32 groups take 0.8 to 1.0 of the time.  (Such rows on 16-byte boundaries stay in
// groups; their last bits may differ from those of other layouts.)
bool minibatch_vec(int64_t d, int32_t B, bool aligned) { return d > 256 || (d % 4 == 0 && (aligned || (d > 64 && B <= 32))); }

// The chunked kernel for rows of d columns.  Workgroup size and column groups per thread are a
// function of d alone and equal those of the one-pass variant for the same d, so either kernel (and
// the fused form) produces the same bits.
template <int FUSE>
static hipError_t launch_chunked(const GemvArgs& g, hipStream_t st) {
  const int64_t d4 = (g.d + 3) / 4;
  const bool odd = g.d % 4 != 0;
  dim3 grid((unsigned)g.n);
#define CECA_CHUNKED(T, CH, G)                                                              \
  do {                                                                                      \
    if (odd) grad_chunked_kernel<4, T, CH, G, FUSE, true><<<grid, dim3(T), 0, st>>>(g);     \
    else grad_chunked_kernel<4, T, CH, G, FUSE, false><<<grid, dim3(T), 0, st>>>(g);        \
  } while (0)
  if (!g.vec) {
    if (g.d <= 64) grad_chunked_kernel<1, 64, 8, 1, FUSE, false><<<grid, dim3(64), 0, st>>>(g);
    else grad_chunked_kernel<1, 256, 8, 1, FUSE, false><<<grid, dim3(256), 0, st>>>(g);
  }
  else if (d4 <= 64) CECA_CHUNKED(64, 8, 1);           // (other wavefronts would add zeros)
  else if (d4 <= 256) CECA_CHUNKED(256, 8, 1);
  else if (d4 <= 1024) CECA_CHUNKED(1024, 8, 1);
  else if (d4 <= 2048) CECA_CHUNKED(1024, 4, 2);
  else CECA_CHUNKED(1024, 2, 4);
#undef CECA_CHUNKED
  return hipGetLastError();
}

// A one-pass variant with the whole batch in registers exists for (B, d4).
static bool onepass_tile_exists(int32_t B, int64_t d4) {
  return (B <= 32 && d4 <= 256) || (B <= 16 && d4 <= 1024) || (B <= 8 && d4 <= 2048) || (B <= 4 && d4 <= 4096);
}

// Where the chunked kernel is the default for a single step (rows of up to 16384 columns, any batch): single columns; many
// agents with long rows, two workgroups per compute unit; and batches for which no register tile exists on rows of up to 1024
// columns, which margins and half step would read twice (n = 746, d = 188, B = 64 29 us per iteration against 15, n = 841, d =
// 528, B = 55 45 against 23, n = 26, d = 250, B = 41 equal).
// How many agents are many, two-pass against chunked, 20 iterations of B = 17 / 32 / 64: n = 96 at d = 2500 284 / 347 / 582
// us against 254 / 325 / 569, at d = 12000 819 / 1197 / - against 651 / 1069; n = 80 at d = 2500 252 / 291 / 449 against 250 /
// 319 / 560; on rows of little more than 1024 columns workgroups are too few for large batches (n = 112, d = 1200 241 / 283 /
// 428 against 215 / 270 / 473).
static bool chunked_by_default(int32_t n, int64_t d, int32_t B, bool vec) {
  const int64_t d4 = (d + 3) / 4;
  if (!vec) return true;
  if (d4 > 4096) return false;
  return d4 <= 256 ? B > 32 : n >= 128 || (n >= 96 && (d > 2048 || B <= 32));
}

// Rows of more than 2048 columns that are no whole groups, on few agents: margins and half step, in 16-byte groups, and windows
// in chunks for batches of up to kTwoPassWindow samples, which single columns had before (where their words fitted the workspace: per
// iteration n = 8, d = 2265, B = 2 3.3 us against 6.9 with two kernels, n = 2, d = 5702, B = 2 3.7 against 6.4).  One workgroup per
// agent is not better throughout (n = 6, d = 2051, B = 9 4.6 us per iteration in a window of such workgroups against 8.0, n = 3, d =
// 9001, B = 4 12.8 with one kernel per iteration against 7.8), and where the line lies has not been measured.  With more
// agents than a window takes the other forms' rules apply (n = 100, d = 2101, B = 16 13.2 -> 10.4).
bool two_pass_rows(int32_t n, int64_t d) { return d % 4 != 0 && d > 2048 && n <= 32; }

// Shapes whose iterations can run as one fused kernel each with the bits of single steps: those where a
// single step already uses the chunked kernel, and those where it uses a one-pass variant (same bits).
// Few agents with a batch too large for a register tile stay with the two-pass kernels: a handful of
// workgroups walking megabytes of rows would be slower than three launches.
bool grad_fused_covers(int32_t n, int64_t d, int32_t B, bool vec) {
  return n >= 2 && (chunked_by_default(n, d, B, vec) || (onepass_tile_exists(B, (d + 3) / 4) && !two_pass_rows(n, d)));
}

bool launch_grad_fused(const GemvArgs& g, hipStream_t st, hipError_t* err) {
  if (!grad_fused_covers(g.n, g.d, g.B, g.vec)) return false;
  *err = launch_chunked<1>(g, st);
  return true;
}

// The same with the state kept in half-step form between iterations (px, py -> ox, oy: two different buffers).
bool launch_grad_half(const GemvArgs& g, hipStream_t st, hipError_t* err) {
  if (!grad_fused_covers(g.n, g.d, g.B, g.vec)) return false;
  if (g.px == g.ox && !g.p_first) { *err = hipErrorInvalidValue; return true; }     // peers' rows are read while rows are written
  *err = launch_chunked<2>(g, st);
  return true;
}

// Batches over 32 on rows of up to 1024 columns, in a step of its own: a workgroup walks them in dependent groups of eight rows,
// where two passes have a workgroup per group, and few agents leave compute units idle.  Two passes against one, step in a captured
// graph: d = 400, B = 64 n = 4 9.9 us against 12.6, n = 128 11.8 against 13.4, n = 256 14.7 against 15.3; B = 40 n = 4 9.0
// against 9.9, n = 96 10.3 against 10.5, n = 128 11.2 against 10.9; d <= 256 (64 threads) B = 64 n = 8 10.0 against 11.1, n = 96
// 11.4 against 11.5, B = 48 9.7 against 9.5, B = 33 9.2 against 8.6.  (Runs fuse one-pass iterations into one kernel each.)
static bool two_passes_alone(const GemvArgs& g) {
  return g.vec && g.d <= 1024 && g.B > 32 && (g.d <= 256 ? g.B > 48 && g.n < 96 : g.n < (g.B > 48 ? 256 : 128));
}

// Picks the one-pass variant whose register tile covers (B, d); false if none does.
bool launch_grad_onepass(const GemvArgs& g, bool alone, hipStream_t st, hipError_t* err) {
  if (alone && two_passes_alone(g)) return false;
  const int64_t d4 = (g.d + 3) / 4;
  const int apw = g_tuning.agents_per_wg;
  // many agents, long rows: the chunked kernel (any B up to 64, d up to 16384), two workgroups per
  // compute unit; a handful of agents cannot fill the device that way and stays with the kernels below
  if (chunked_by_default(g.n, g.d, g.B, g.vec) && (!g_tuning.never_chunked || !g.vec)) {
    *err = launch_chunked<0>(g, st);
    return true;
  }
  if (two_pass_rows(g.n, g.d)) return false;
  // Rows of odd length where the looping kernel requests more than the batch (16 rows for one to eight, d <= 1024: a step 0.96 of the
  // time, d = 385 6.7 us -> 6.4) or its tile spills (d > 8192, four groups per thread; n = 40, d = 9001, B = 2 19 -> 11 us).
  if (g.d % 4 != 0 && !g_tuning.never_chunked && apw == 0 && (d4 <= 256 ? g.B <= 8 : d4 > 2048 && g.B <= 4)) {
    *err = launch_chunked<0>(g, st);
    return true;
  }
  // 1024-thread workgroups fill a compute unit alone: one per unit, each looping over its agents;
  // 256-thread workgroups leave room for several per unit
#define CECA_ONEPASS(T, BM, GG)                                          \
  if (g.B <= BM && d4 <= (int64_t)T * GG) {                              \
    const int per_wg = apw > 0 ? apw : (T == 1024 ? (g.n + 255) / 256 : 1); \
    dim3 grid((unsigned)((g.n + per_wg - 1) / per_wg));                  \
    if (g.d % 4) grad_onepass_kernel<T, BM, GG, true><<<grid, dim3(T), 0, st>>>(g); \
    else grad_onepass_kernel<T, BM, GG, false><<<grid, dim3(T), 0, st>>>(g); \
    *err = hipGetLastError();                                            \
    return true;                                                         \
  }
  CECA_ONEPASS(64, 16, 1)                  // (other wavefronts would add zeros)
  CECA_ONEPASS(64, 32, 1)
  CECA_ONEPASS(256, 16, 1)
  CECA_ONEPASS(256, 32, 1)
  CECA_ONEPASS(1024, 8, 1)
  CECA_ONEPASS(1024, 16, 1)
  CECA_ONEPASS(1024, 8, 2)
  CECA_ONEPASS(1024, 4, 4)
#undef CECA_ONEPASS
  return false;
}

// A whole iteration of a small problem in one launch.  The gradient kernel and the combine cost a launch each (about
// 5 us) at sizes whose work takes one or two, and what separates them is that the combine needs a peer's message.  Here
// a workgroup of 2 x THREADS threads evaluates two messages side by side: the first half its own agent's, the second
// half that agent's peer's, which passes through LDS.  With one port the two are each other's peers, so a workgroup
// finishes both (also in place); with two ports every gradient is taken twice, and the rule in launch_pair_step keeps
// to problems whose rows cost less than the launch saved.
// Arithmetic and order of summation: the one-pass kernels' and the combine kernel's, operation for operation.
template <int VEC, int THREADS, int BMAX>
__global__ __launch_bounds__(2 * THREADS) void pair_step_kernel(const GemvArgs P) {
  using V = typename VecOf<VEC>::T;
  constexpr int WAVES = THREADS / 64;
  constexpr int CH = kRowGroup;
  constexpr int MG = BMAX < 16 ? BMAX : 16;            // samples per wavefront sum (any number gives the same bits)
  __shared__ float red[2][WAVES][BMAX];
  __shared__ V msg_s[2][THREADS];
  const int tid = threadIdx.x % THREADS, lane = threadIdx.x & 63;
  const int half = __builtin_amdgcn_readfirstlane((int)threadIdx.x / THREADS);        // the same for a whole wavefront
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool both = P.p_port == 1;                     // an even agent and the odd one it is paired with (Eq. (7))
  const int first = both ? 2 * (int)blockIdx.x : (int)blockIdx.x;
  int p;
  if (both) {
    p = first + P.p_shift; if (p >= P.n) p -= P.n;
  } else {
    p = first - P.p_shift; if (p < 0) p += P.n;
  }
  const int agent = half ? p : first;
  const int64_t c = (int64_t)tid * VEC;
  const bool on = c < P.d;                             // d is a multiple of VEC
  const int64_t col = on ? c : 0;
  // lane j holds sample j; samples past B repeat the last
  const int32_t myidx = min(max(P.batch_idx[(int64_t)agent * P.B + min(lane, P.B - 1)], 0), P.N - 1);
  const float tmine = P.t[(int64_t)agent * P.N + myidx];
  const float* Abase = P.A + (int64_t)agent * P.N * P.lda + col;
  V a[BMAX];
#pragma unroll
  for (int j = 0; j < BMAX; ++j) a[j] = V(0.0f);       // groups past B are never requested
#pragma unroll
  for (int c0 = 0; c0 < BMAX; c0 += CH) {
    if (c0 < P.B) {
#pragma unroll
      for (int j = c0; j < c0 + CH; ++j) a[j] = ld_plain<V>(Abase + (int64_t)__builtin_amdgcn_readlane(myidx, j) * P.lda);
    }
  }
  const int64_t off = (int64_t)agent * P.ld + col;
  const V x = ld_plain<V>(P.px + off);
  const V y = P.p_read_y || P.p_exch_y ? ld_plain<V>(P.py + off) : V(0.0f);
  const V z = on ? (P.p_exch_y ? y : x) : V(0.0f);
#pragma unroll
  for (int c0 = 0; c0 < BMAX; c0 += MG) {
    float m[MG];
#pragma unroll
    for (int j = 0; j < MG; ++j) m[j] = dot_v(a[c0 + j], z);
    int jrow;
    bool owner;
    const float msum = wave_sum_many<MG>(m, lane, jrow, owner);
    if (owner) red[half][wave][c0 + jrow] = msum;
  }
  __syncthreads();
  float mj = 0.0f;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) mj += red[half][w][min(lane, BMAX - 1)];
  const float cmine = lane < P.B ? loss_coef(P.kind, mj, tmine, P.scale) : 0.0f;
  V e = V(0.0f);
#pragma unroll
  for (int c0 = 0; c0 < BMAX; c0 += CH) {
    if (c0 < P.B) {
#pragma unroll
      for (int j = c0; j < c0 + CH; ++j) {
        const float cj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cmine), j));
        e += cj * a[j];
      }
    }
  }
  if (P.noise_std != 0.0f) e = add_noise<V>(e, P.noise_std, col, noise_keys(P.seed, P.k, (uint32_t)agent));
  const V v = z - P.lr * e;
  msg_s[half][tid] = v;
  __syncthreads();
  if ((half && !both) || !on) return;
  {
#pragma clang fp contract(off)
    const V msg = msg_s[half ^ 1][tid];
    const V dz = v - z;                                // -lr e
    const V xs = P.p_exch_y ? x + dz : v;
    const V ys = P.p_exch_y ? v : y + dz;
    const int64_t oo = (int64_t)agent * P.ldo + col;
    st_plain<V>(P.ox + oo, combine(P.pa, xs, P.pap, msg));
    st_plain<V>(P.oy + oo, P.p_read_y ? combine(P.pb, ys, P.pbp, msg) : P.pbp * msg);
  }
}

// Where the pair form applies: rows that one 64- or 256-thread workgroup takes in one pass, and few enough of them --
// 8 MB in all, 1.5 us of streaming, twice -- that taking every gradient twice costs less than a launch.  Per step in a
// captured graph, two kernels against this one: n = 6, d = 1000, B = 8: 6.4 -> 3.2 us; n = 258, d = 10, B = 50: 9.3 ->
// 5.4 (one port 4.6); and at the limit n = 64, d = 1024, B = 32: 7.8 -> 5.7 (one port 5.6); n = 2000, d = 64, B = 16: 12.3 -> 5.5; n = 4000,
// d = 10, B = 50: 18.2 -> 14.6.
bool launch_pair_step(const GemvArgs& g, hipStream_t st, hipError_t* err) {
  const bool both = g.p_port == 1, vec4 = g.vec;
  if ((int64_t)g.n * g.B * g.d * 4 > (8LL << 20)) return false;
  if (g.d % 4 != 0 && g.d > 256) return false;       // pair_step_kernel has no instructions for a short last group, and single columns end at 256
  if (both ? (g.n & 1) || !(g.p_shift & 1) : g.px == g.ox) return false;       // two ports: out of place only
  const dim3 grid((unsigned)(both ? g.n / 2 : g.n));
#define CECA_PAIR(VEC, T, BM)                                                \
  if (vec4 == (VEC == 4) && g.d <= (int64_t)T * VEC && g.B <= BM) {          \
    pair_step_kernel<VEC, T, BM><<<grid, dim3(2 * T), 0, st>>>(g);           \
    *err = hipGetLastError();                                                \
    return true;                                                             \
  }
  CECA_PAIR(4, 64, 8)                      // (the 256-thread kernels' other wavefronts would add zeros)
  CECA_PAIR(4, 64, 16)
  CECA_PAIR(4, 64, 32)
  CECA_PAIR(4, 256, 8)
  CECA_PAIR(4, 256, 16)
  CECA_PAIR(4, 256, 32)
  CECA_PAIR(1, 64, 16)
  CECA_PAIR(1, 64, 64)
  CECA_PAIR(1, 256, 16)
  CECA_PAIR(1, 256, 64)
#undef CECA_PAIR
  return false;
}

hipError_t launch_margins(const GemvArgs& g, hipStream_t st) {
  if (g.nchunks < 1 || g.n > 65535) return hipErrorInvalidConfiguration;
  dim3 grid((unsigned)g.nchunks, (unsigned)g.n, (unsigned)((g.B + kRowGroup - 1) / kRowGroup)), block(kBlock);
  if (!g.vec) margins_kernel<1, false, false><<<grid, block, 0, st>>>(g);
  else if (g.d % 4) margins_kernel<4, true, false><<<grid, block, 0, st>>>(g);
  else margins_kernel<4, false, false><<<grid, block, 0, st>>>(g);
  return hipGetLastError();
}

hipError_t launch_margins_fused(const GemvArgs& g, hipStream_t st) {
  if (g.nchunks < 1 || g.n > 65535) return hipErrorInvalidConfiguration;
  // the row groups of an (agent, chunk) pair all read the old rows while the first one stores the new ones
  if (g.px == g.ox || g.py == g.oy) return hipErrorInvalidValue;
  dim3 grid((unsigned)g.nchunks, (unsigned)g.n, (unsigned)((g.B + kRowGroup - 1) / kRowGroup)), block(kBlock);
  if (!g.vec) margins_kernel<1, false, true><<<grid, block, 0, st>>>(g);
  else if (g.d % 4) margins_kernel<4, true, true><<<grid, block, 0, st>>>(g);
  else margins_kernel<4, false, true><<<grid, block, 0, st>>>(g);
  return hipGetLastError();
}

hipError_t launch_halfstep(const GemvArgs& g, hipStream_t st) {
  const int vec = g.vec ? 4 : 1;
  const int64_t groups = (g.d + vec - 1) / vec;
  const int64_t gx = (groups + kBlock - 1) / kBlock;
  if (gx < 1 || gx > 0x7fffffffLL || g.n > 65535) return hipErrorInvalidConfiguration;
  dim3 grid((unsigned)gx, (unsigned)g.n), block(kBlock);
  if (!g.vec) halfstep_kernel<1, false><<<grid, block, 0, st>>>(g);
  else if (g.d % 4) halfstep_kernel<4, true><<<grid, block, 0, st>>>(g);
  else halfstep_kernel<4, false><<<grid, block, 0, st>>>(g);
  return hipGetLastError();
}

}  // namespace ceca
