// A whole window of minibatch iterations in one kernel, for problems small enough that every workgroup is resident
// at once (see dsgd_ceca_run in ceca.h).
#include <hip/hip_runtime.h>

#include "ceca.h"
#include "device_util.h"
#include "gemv_util.h"
#include "launch.h"

namespace ceca {

// ---------------------------------------------------------------------------------------------
// One launch per iteration costs 4.5 to 14 us at sizes whose arithmetic takes a fraction of that.  Here a workgroup
// owns one agent's columns (all of them, or one chunk of 256 threads' columns where the gradient of a single step
// takes two passes) and keeps x and y in registers for the whole call; what has to cross workgroups -- an agent's
// message, and the partial margins of a chunk -- goes through memory as 8-byte words {tag, value}, written and
// polled with device-scope atomics.  The tag (iteration + 1) arrives with its value, so an exchange is one store and
// one load that sees it: no flags, fences or cache write-backs.
//
// Slots alternate between two iterations.  A message slot is written again two iterations later, after the agent
// that read it has been seen to publish the iteration in between (it consumed the old message before that); the
// partial margins need no such look, because a workgroup takes the next iteration's margins from every chunk of its
// agent, and each of those published them after it had consumed the old ones.
// Every wait is for something published one iteration earlier, or for this iteration's words of workgroups that wait
// only on earlier ones: once every workgroup is on the device every wait ends.  The host's rule makes that likely but
// cannot promise it (other processes, replays of a captured call on a narrower stream), so one more workgroup calls the
// roll: when it has seen the first words of every other it marks the window as complete.  A workgroup that has waited for
// kRollCallPolls polls while it is not complete marks it as given up.  Both are a compare-and-swap on one word that is
// zero before, so the window is one or the other for good, the same for everybody.  Results are stored only by a
// complete window.  From one given up the workgroups leave as they come to the end, and the last one to leave does
// the whole window alone (run_alone), from the untouched state and with the same bits.  The others pay a look at that
// word after their last exchange (requested inside the loop it costs every iteration 0.4 us: the compiler waits for it
// before the next rows' requests).  With a count that every workgroup adds itself to, the atomics on one word took 3 us of
// a call with 426 agents, 73 -> 76 us.
//
// What bounds it: the latency of the chain rows -> margins -> barrier -> coefficients -> message -> peer, once per
// iteration (a store and the load that sees it take 0.83 us between two workgroups on different XCDs, 0.58 us on one), and
// a compute unit's intake of sampled rows, 75 GB/s.
// Per iteration, one launch (two in chunks) each before and here: n = 5, d = 1000, B = 8: 3.9 -> 1.9 us, on one XCD 1.7; n = 258, d = 10,
// B = N = 50 with noise: 7.6 -> 2.5 us; n = 6, d = 10000, B = 32 in ten chunks: 13.4 -> 5.9 us; n = 256, d = 256, B = 32:
// 8.4 -> 2.6 us.
// Messages packed as four floats in three words were slower (n = 5: 2.2 -> 2.5 us in the same loop), and 128-thread
// workgroups with a margin word per wavefront too (n = 6, d = 10000, B = 32: 5.9 -> 6.6 us: four times the polling).
//
// Arithmetic and order of summation are those of the single-step kernels (gemv.hip), operation for operation: per
// sample the dot product over a thread's columns, the wavefront butterfly 8 samples at a time, wavefronts in order,
// then chunks in order.
// ---------------------------------------------------------------------------------------------
typedef unsigned long long Word;

// Waits are counted in polls, a quarter of a microsecond each: they stand still while the process is off the device.
// 12 ms: what a window done alone takes (n = 5, d = 1000, B = 8, 200 iterations: 2 ms; n = 258, d = 10, B = 50, 20
// iterations: 40 ms; n = 6, d = 10000, B = 32, 100 iterations: 46 ms).
constexpr uint32_t kRollCallPolls = 64 * 1024;
// In a complete window no wait lasts; this bound is for a workspace that something else writes to during the call: NaN
// takes the place of what never came, and the call ends.
constexpr uint32_t kGiveUpPolls = 128 * 1024 * 1024;             // half a minute
constexpr uint32_t kLost = 1u << 31;
// the word of the roll: its two marks, and a count of the workgroups that left a window given up (bits 32 to 62)
constexpr Word kComplete = 1, kLeft = 1ULL << 32, kGivenUp = 1ULL << 63;

__device__ __forceinline__ Word peek(const Word* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void publish(Word* p, uint32_t tag, float v) {
  __hip_atomic_store(p, ((Word)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A bounded wait: false once the window has been given up, then for good.
struct Patience {
  Word* roll;
  uint32_t polls = 0;                      // of this wait; from kLost on: given up
  __device__ __forceinline__ Patience(const RunArgs& P) : roll(P.roll) {}
  __device__ __forceinline__ void begin() { polls &= kLost; }
  __device__ __forceinline__ bool again() {
    if ((++polls & 1023u) == 0 && hopeless()) polls = kLost;
    return polls < kLost;
  }
  __device__ __forceinline__ bool hopeless() {
    Word w = peek(roll);
    if (w & kGivenUp) return true;
    if (w & kComplete) return polls >= kGiveUpPolls;
    // fails if the word has changed meanwhile: then the next look decides
    return polls >= kRollCallPolls && settle(roll, kGivenUp);
  }
  static __device__ __forceinline__ bool settle(Word* roll, Word mark) {
    Word w = 0;
    return __hip_atomic_compare_exchange_strong(roll, &w, mark, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // waits for one of the marks, from word w on; true if the window is complete
  __device__ __forceinline__ bool complete(Word w) {
    begin();
    while (!(w & (kComplete | kGivenUp))) {
      (void)again();
      w = peek(roll);
    }
    return !(w & kGivenUp);
  }
};

template <int VEC> struct Parts;
template <> struct Parts<1> {
  static __device__ __forceinline__ float get(float v, int) { return v; }
  static __device__ __forceinline__ void set(float& v, int, float f) { v = f; }
};
template <> struct Parts<4> {
  static __device__ __forceinline__ float get(vf4 v, int u) { return v[u]; }
  static __device__ __forceinline__ void set(vf4& v, int u, float f) { v[u] = f; }
};

// wavefronts per SIMD the kernel is compiled for (the host's residency rule counts on them): BMAX rows of VEC
// columns and about 70 more registers per thread, nothing spilled to memory (scalar registers go to spare vector registers)
template <int VEC, int THREADS, int BMAX>
constexpr int run_waves() { return THREADS == 1024 || VEC == 1 || BMAX <= 8 ? 4 : BMAX <= 16 ? 3 : BMAX <= 32 ? 2 : 1; }

// Whose message an agent reads (Eqs. (6), (7)).
__device__ __forceinline__ int peer_of(const RunArgs& P, const MultiRound& R, int agent) {
  int p = P.port == 2 || (agent & 1) ? agent - R.shift : agent + R.shift;
  if (p < 0) p += P.n;
  if (p >= P.n) p -= P.n;
  return p;
}

// Words of an agent's message (RunArgs::dw; rows of whole groups have as many as columns: one number fewer in scalar registers).
template <bool ODD> __device__ __forceinline__ int64_t row_words(const RunArgs& P) { return ODD ? P.dw : P.d; }

// The whole window by one workgroup: iteration by iteration every agent's message, then every agent's combine, with the
// state in the output rows and the messages in the workspace.  Operation for operation what the workgroups of run_kernel
// do together; `red` and `part` are theirs.
template <int VEC, int THREADS, int BMAX, bool CHUNKS, bool ODD>
__device__ __forceinline__ void run_alone(const RunArgs& P, float (&red)[2][THREADS / 64][BMAX], float* part) {
  using V = typename VecOf<VEC>::T;
  constexpr int WAVES = THREADS / 64;
  constexpr int CH = kRowGroup;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));                                  // nothing derived from it waits in run_kernel's registers
  const int lane = tid & 63, wave = tid >> 6;
  float* msgs = reinterpret_cast<float*>(P.words);               // n rows of `pitch`: whole groups
  const int64_t pitch = (P.d + VEC - 1) / VEC * VEC;
  int r = P.r0;
  for (int t = 0; t < P.iters; ++t) {
    const MultiRound& R = P.round[r];
    const float* xin = t == 0 ? P.xin : P.xout;
    const float* yin = t == 0 ? P.yin : P.yout;
    const float* zin = R.exch_y ? yin : xin;
    for (int agent = 0; agent < P.n; ++agent) {
      const int32_t myidx = min(max(P.batch_idx[((int64_t)t * P.n + agent) * P.B + min(lane, P.B - 1)], 0), P.N - 1);
      const float tmine = P.t[(int64_t)agent * P.N + myidx];
      const float* Abase = P.A + (int64_t)agent * P.N * P.lda;
      float mj = 0.0f;
      for (int chunk = 0; chunk < P.nchunks; ++chunk) {
        const int64_t first = (int64_t)chunk * THREADS * VEC, c = first + tid * VEC;
        const bool on = c < P.d;
        const int back = on ? short_back<ODD>(c, P.d) : 0;
        const V zr = on ? last_columns(ld_own<V>(zin + (int64_t)agent * P.ld + c, back), back) : V(0.0f);
        for (int c0 = 0; c0 < P.B; c0 += CH) {
          float m[CH];
#pragma unroll
          for (int j = 0; j < CH; ++j)
            m[j] = dot_v(own_of_row(ld_plain<V>(Abase + (int64_t)__builtin_amdgcn_readlane(myidx, c0 + j) * P.lda + (on ? c - back : first)), ODD ? columns_left(c, P.d) : 4), zr);
          int jrow;
          bool owner;
          const float msum = wave_sum_many<CH>(m, lane, jrow, owner);
          if (owner) red[0][wave][c0 + jrow] = msum;
        }
        __syncthreads();
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) s += red[0][w][min(lane, P.B - 1)];
        if (!CHUNKS) mj = s;
        else if (tid < P.B) part[chunk * P.B + tid] = s;
        __syncthreads();
      }
      if (CHUNKS)
        for (int ch = 0; ch < P.nchunks; ++ch) mj += part[ch * P.B + min(lane, P.B - 1)];
      const float cmine = lane < P.B ? loss_coef(P.kind, mj, tmine, P.scale) : 0.0f;
      for (int chunk = 0; chunk < P.nchunks; ++chunk) {
        const int64_t first = (int64_t)chunk * THREADS * VEC, c = first + tid * VEC;
        const bool on = c < P.d;
        const int back = on ? short_back<ODD>(c, P.d) : 0;
        const V z = on ? ld_own<V>(zin + (int64_t)agent * P.ld + c, back) : V(0.0f);
        V e = V(0.0f);
        for (int c0 = 0; c0 < P.B; c0 += CH) {
#pragma unroll
          for (int j = 0; j < CH; ++j) {
            const V a = ld_plain<V>(Abase + (int64_t)__builtin_amdgcn_readlane(myidx, c0 + j) * P.lda + (on ? c - back : first));
            const float cj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cmine), c0 + j));
            e += cj * a;
          }
        }
        e = own_columns(e, back);
        if (P.noise_std != 0.0f) e = add_noise<V>(e, P.noise_std, on ? c : 0, noise_keys(P.seed, P.k + (uint32_t)t, (uint32_t)agent));
        const V v = z - P.lr * e;
        if (on) *reinterpret_cast<V*>(msgs + (int64_t)agent * pitch + c) = v;
      }
    }
    __syncthreads();
    for (int agent = 0; agent < P.n; ++agent) {
      const int p = peer_of(P, R, agent);
      for (int64_t c = (int64_t)tid * VEC; c < P.d; c += (int64_t)THREADS * VEC) {
#pragma clang fp contract(off)
        const int64_t off = (int64_t)agent * P.ld + c;
        const int back = short_back<ODD>(c, P.d);
        const V x = ld_own<V>(xin + off, back), y = ld_own<V>(yin + off, back), z = R.exch_y ? y : x;
        const V v = ld_plain<V>(msgs + (int64_t)agent * pitch + c), msg = ld_plain<V>(msgs + (int64_t)p * pitch + c);
        const V dz = v - z;
        const V xs = R.exch_y ? x + dz : v;
        const V ys = R.exch_y ? v : y + dz;
        st_own<V>(P.xout + off, combine(R.a, xs, R.ap, msg), back);
        st_own<V>(P.yout + off, R.read_y ? combine(R.b, ys, R.bp, msg) : R.bp * msg, back);
      }
    }
    __syncthreads();
    r = r + 1 == P.tau ? 0 : r + 1;
  }
}

// The roll: a workgroup is there when its first word has a tag -- the margin of sample 0 of its chunk, or the first word
// of its agent's message.  True if the window is complete.
template <int THREADS, bool CHUNKS, bool ODD>
__device__ __forceinline__ bool call_roll(const RunArgs& P) {
  Patience wait(P);
  bool here = true;
  for (int i = threadIdx.x; i < P.n * P.nchunks && here; i += THREADS) {
    const Word* first = P.words + (CHUNKS ? 2 * (int64_t)P.n * row_words<ODD>(P) + (int64_t)i * P.B : (int64_t)i * row_words<ODD>(P));
    wait.begin();
    do here = (peek(first) >> 32) != 0;
    while (!here && wait.again());
  }
  if (__syncthreads_and(here) && threadIdx.x == 0) (void)Patience::settle(P.roll, kComplete);
  return wait.complete(0);
}

// Workgroup `wg`'s part of the window.  True if the window is complete and the results are stored.
template <int VEC, int THREADS, int BMAX, bool CHUNKS, bool ODD>
__device__ __forceinline__ bool take_part(const RunArgs& P, int wg, float (&red)[2][THREADS / 64][BMAX], float* part) {
  using V = typename VecOf<VEC>::T;
  constexpr int WAVES = THREADS / 64;
  constexpr int CH = kRowGroup;            // rows are requested and added up in groups, as in the single-step kernels
  constexpr int MG = BMAX < 16 ? BMAX : 16;    // samples per wavefront sum (any number gives the same bits)
  static_assert(BMAX % CH == 0 && BMAX <= 64, "whole groups of samples, one lane per sample");
  const int agent = CHUNKS ? (int)((uint32_t)wg / (uint32_t)P.nchunks) : wg;
  const int chunk = CHUNKS ? (int)((uint32_t)wg % (uint32_t)P.nchunks) : 0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // lanes past the last column carry z = 0; they publish and wait for nothing
  const int64_t c = ((int64_t)chunk * THREADS + tid) * VEC;
  const bool on = c < P.d;
  const int64_t col = on ? c : 0;
  const int back = short_back<ODD>(col, P.d);
  // message words of an agent: VEC planes of a word per group, so that neighbouring lanes touch neighbouring words
  // (all of a window's words are far fewer than 2^31)
  const uint32_t words = (uint32_t)row_words<ODD>(P), plane = words / VEC, group = (uint32_t)col / VEC;

  V x = ld_own<V>(P.xin + (int64_t)agent * P.ld + col, back);
  V y = ld_own<V>(P.yin + (int64_t)agent * P.ld + col, back);
  // a row's address is the agent's base in scalar registers plus 32 bits (the host sees to it that they are enough):
  // the row's distance, computed once per batch in lane j for sample j, and the thread's own offset
  const int lead = ODD && chunk > 0 ? 16 : 0;
  const char* Abase = reinterpret_cast<const char*>(P.A + (int64_t)agent * P.N * P.lda + (int64_t)chunk * THREADS * VEC) - lead;
  // lanes past the last column read the chunk's first one; a short last group that opens a chunk starts before it
  const uint32_t voff = (uint32_t)(lead + (on ? (tid * VEC - back) * 4 : 0));
  const float* tbase = P.t + (int64_t)agent * P.N;
  const int32_t* idx = P.batch_idx + (int64_t)agent * P.B + min(lane, P.B - 1);    // samples past B repeat the last
  const int64_t nb = (int64_t)P.n * P.B;
  int32_t myidx = min(max(idx[0], 0), P.N - 1);
  V a[BMAX];
#pragma unroll
  for (int j = 0; j < BMAX; ++j) a[j] = V(0.0f);      // groups past B are never requested
  float tmine;
  const bool short_wave = ODD && __any(back != 0);           // rows are not moved for a short last group: see z_for_rows
  auto request_rows = [&]() {
    tmine = tbase[myidx];
    const uint32_t dist = (uint32_t)myidx * (uint32_t)P.lda * (uint32_t)sizeof(float);
#pragma unroll
    for (int c0 = 0; c0 < BMAX; c0 += CH) {
      if (c0 < P.B) {                      // the same for every thread
#pragma unroll
        for (int j = c0; j < c0 + CH; ++j)
          a[j] = ld_plain<V>(reinterpret_cast<const float*>(Abase + (voff + (uint32_t)__builtin_amdgcn_readlane((int)dist, j))));
      }
    }
  };
  request_rows();
  // the next batch's numbers: a pointer moved on, or, where that costs, worked out anew each time (single columns in 256 threads with 64 rows,
  // per 36 iterations: n = 40, d = 199, B = 46 102.5 us against 98.7, n = 125, d = 255, B = 64 112.6 against 107.7; elsewhere the pointer
  // is 1 to 2 % ahead, n = 258, d = 10, B = 50 93.0 against 94.4)
  constexpr bool INDEXED = VEC == 1 && THREADS == 256 && BMAX == 64;
  if (!INDEXED) idx += P.iters > 1 ? nb : 0;
  int32_t idx_next = INDEXED ? idx[P.iters > 1 ? nb : 0] : *idx;
  Patience wait(P);
  int r = P.r0;
  int reader = agent;                      // who read my message two iterations ago (after the shifts below)
  int reader1 = agent;                     // and one iteration ago
  for (int t = 0; t < P.iters; ++t) {
    const int par = t & 1;
    const MultiRound& R = P.round[r];
    const uint32_t tag = (uint32_t)t + 1;
    const int p = peer_of(P, R, agent);    // whose message I read, and who reads mine
    int to = p;
    if (P.port == 2) { to = agent + R.shift; if (to >= P.n) to -= P.n; }
    // the look at the reader of my message of iteration t - 2: has it published iteration t - 1?
    const Word* seen = P.words + ((uint32_t)((par ^ 1) * P.n + reader) * words + group);
    Word ack = 0;
    if (t >= 2 && on) ack = peek(seen);

    const V z = on ? (R.exch_y ? y : x) : V(0.0f);
    const V zr = short_wave ? last_columns(z, back) : z;
    // every group of the tile, also those past B (zeros): without branches the groups' chains overlap
#pragma unroll
    for (int c0 = 0; c0 < BMAX; c0 += MG) {
      float m[MG];
#pragma unroll
      for (int j = 0; j < MG; ++j) m[j] = dot_v(a[c0 + j], zr);
      if (ODD && some_nan(m)) {
#pragma unroll
        for (int j = 0; j < MG; ++j) m[j] = dot_v(own_of_row(a[c0 + j], columns_left(c, P.d)), zr);
      }
      int jrow;
      bool owner;
      const float msum = wave_sum_many<MG>(m, lane, jrow, owner);
      if (owner) red[par][wave][c0 + jrow] = msum;
    }
    __syncthreads();
    float mj = 0.0f;
    if (CHUNKS) {
      Word* ring = P.words + (2 * (uint32_t)P.n * words + (uint32_t)(par * P.n + agent) * (uint32_t)(P.nchunks * P.B));
      if (tid < P.B) {
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) s += red[par][w][tid];
        publish(ring + chunk * P.B + tid, tag, s);
      }
      const int count = P.nchunks * P.B;   // at most kRunParts
      for (int i0 = tid; i0 < count; i0 += 2 * THREADS) {
        const int i1 = min(i0 + THREADS, count - 1);             // two words in flight; past the end the last one again
        Word w0, w1;
        bool here;
        wait.begin();
        do {
          w0 = peek(ring + i0);
          w1 = peek(ring + i1);
          here = (uint32_t)(w0 >> 32) == tag && (uint32_t)(w1 >> 32) == tag;
        } while (!here && wait.again());
        part[i0] = here ? __uint_as_float((uint32_t)w0) : __builtin_nanf("");
        part[i1] = here ? __uint_as_float((uint32_t)w1) : __builtin_nanf("");
      }
      __syncthreads();
      const int j = min(lane, P.B - 1);
      int ch = 0;                          // four words of LDS on their way at a time, added in order (490 -> 485 us in ten chunks)
      for (; ch + 4 <= P.nchunks; ch += 4) {
        float q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = part[(ch + u) * P.B + j];
#pragma unroll
        for (int u = 0; u < 4; ++u) mj += q[u];
      }
      for (; ch < P.nchunks; ++ch) mj += part[ch * P.B + j];
    } else {
      const int j = min(lane, BMAX - 1);
#pragma unroll
      for (int w = 0; w < WAVES; ++w) mj += red[par][w][j];
    }
    // every wavefront turns the margins into coefficients for itself (lane j: sample j)
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
    if (short_wave) e = own_columns(e, back);
    if (P.noise_std != 0.0f) e = add_noise<V>(e, P.noise_std, col, noise_keys(P.seed, P.k + (uint32_t)t, (uint32_t)agent));
    const V v = z - P.lr * e;

    if (t >= 2 && on) {
      wait.begin();
      while ((uint32_t)(ack >> 32) < (uint32_t)t && wait.again()) ack = peek(seen);
    }
    if (on) {
      Word* slot = P.words + ((uint32_t)(par * P.n + agent) * words + group);
#pragma unroll
      for (int u = 0; u < VEC; ++u) publish(slot + u * plane, tag, Parts<VEC>::get(v, u));
    }
    // the next iteration's rows travel while the message does; a batch of the same rows (full gradients) is there
    if (t + 1 < P.iters) {
      const int32_t now = myidx;
      myidx = min(max(idx_next, 0), P.N - 1);
      if (__any(now != myidx)) request_rows();                   // the same in every wavefront
      if (!INDEXED) idx += t + 2 < P.iters ? nb : 0;
      idx_next = INDEXED ? idx[(int64_t)min(t + 2, P.iters - 1) * nb] : *idx;
    }
    V msg = V(0.0f);
    if (on) {
      const Word* slot = P.words + ((uint32_t)(par * P.n + p) * words + group);
      wait.begin();
      Word w[VEC];
      bool here;
      do {
        here = true;
#pragma unroll
        for (int u = 0; u < VEC; ++u) w[u] = peek(slot + u * plane);
#pragma unroll
        for (int u = 0; u < VEC; ++u) here = here && (uint32_t)(w[u] >> 32) == tag;
      } while (!here && wait.again());
#pragma unroll
      for (int u = 0; u < VEC; ++u)
        Parts<VEC>::set(msg, u, here ? __uint_as_float((uint32_t)w[u]) : __builtin_nanf(""));
    }
    {
#pragma clang fp contract(off)
      const V dz = v - z;                  // -lr e as the other variable sees it
      const V xs = R.exch_y ? x + dz : v;
      const V ys = R.exch_y ? v : y + dz;
      x = combine(R.a, xs, R.ap, msg);
      y = R.read_y ? combine(R.b, ys, R.bp, msg) : R.bp * msg;
    }
    reader = reader1;
    reader1 = to;
    r = r + 1 == P.tau ? 0 : r + 1;
  }
  if (!wait.complete(peek(P.roll))) return false;                // marked long ago, as a rule
  if (on) {
    st_own<V>(P.xout + (int64_t)agent * P.ld + col, x, back);
    st_own<V>(P.yout + (int64_t)agent * P.ld + col, y, back);
  }
  return true;
}

// ONE_XCD is a template parameter because the chunked instances are at the limit of their scalar registers.
template <int VEC, int THREADS, int BMAX, bool CHUNKS, bool ODD, bool ONE_XCD>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(run_waves<VEC, THREADS, BMAX>(), 8)))
void run_kernel(const RunArgs P) {
  __shared__ float red[2][THREADS / 64][BMAX];                   // alternating between iterations
  __shared__ float part[CHUNKS ? kRunParts : 1];                 // partial margins of every chunk of the agent
  // workgroups go round-robin over the XCDs: of a window on one of them, only every eighth plays
  if (ONE_XCD && (blockIdx.x & 7) != (uint32_t)P.xcd) return;
  const int wg = (int)(ONE_XCD ? blockIdx.x >> 3 : blockIdx.x), wgs = (int)(ONE_XCD ? gridDim.x >> 3 : gridDim.x);
  if (wg + 1 == wgs ? call_roll<THREADS, CHUNKS, ODD>(P) : take_part<VEC, THREADS, BMAX, CHUNKS, ODD>(P, wg, red, part)) return;
  // given up (the same for every thread): nothing has been stored; my own words are behind me before I leave
  __shared__ bool last_s;
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) last_s = (uint32_t)((__hip_atomic_fetch_add(P.roll, kLeft, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ~kGivenUp) >> 32) + 1 == (uint32_t)wgs;
  __syncthreads();
  if (!last_s) return;
  __threadfence();
  run_alone<VEC, THREADS, BMAX, CHUNKS, ODD>(P, red, part);
}

// No word may carry a tag of this call before it is published.
__global__ __launch_bounds__(kBlock) void run_clear_kernel(Word* words, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < count) words[i] = 0;
}

// Threads per workgroup, register rows and chunks for this problem; threads = 0 where the kernel does not apply.
// The shapes are those whose single step sums in the same order: one workgroup per agent where the gradient is taken
// in one pass with one column group per thread, chunks of 256 threads where it takes two passes.
static RunShape run_shape(int32_t n, int64_t d, int32_t B, bool vec4) {
  RunShape s{vec4, 0, 0, 1, 0, false};
  const bool two_pass = vec4 && two_pass_rows(n, d);
  if (n < 2 || B < 1 || B > 64 || (two_pass && B > kTwoPassWindow)) return s;
  const int64_t groups = vec4 ? (d + 3) / 4 : d;
  if (vec4) {
    if (groups <= 64) s.threads = 64;                            // (the single step's other wavefronts add zeros)
    else if (groups <= 256) s.threads = 256;
    else if (two_pass) s.threads = 256;
    else if (groups <= 1024 && B <= 16) s.threads = 1024;
    else if (grad_fused_covers(n, d, B, true)) return s;               // wider rows in one workgroup
    else s.threads = 256;
  } else {
    s.threads = groups <= 64 ? 64 : 256;
  }
  const int64_t chunks = (groups + s.threads - 1) / s.threads;
  if (chunks * B > kRunParts && chunks > 1) return RunShape{vec4, 0, 0, 1, 0, false};
  s.nchunks = (int32_t)chunks;
  s.bmax = vec4 ? (B <= 8 ? 8 : B <= 16 ? 16 : B <= 32 ? 32 : 64) : (B <= 16 ? 16 : 64);
  const int waves = s.threads == 1024 || !vec4 || s.bmax <= 8 ? 4 : s.bmax <= 16 ? 3 : s.bmax <= 32 ? 2 : 1;     // run_waves
  s.wg_per_cu = 4 * waves / (s.threads / 64);
  return s;
}

// Words of an agent's message: whole groups.
static int64_t run_row_words(const RunShape& s, int64_t d) { return s.vec ? (d + 3) / 4 * 4 : d; }

int64_t run_kernel_words(const RunShape& s, int32_t n, int64_t d, int32_t B) {
  return 2 * (int64_t)n * run_row_words(s, d) + (s.nchunks > 1 ? 2 * (int64_t)n * s.nchunks * B : 0);
}

// Every workgroup of the kernel should be resident, whatever else runs (else the window is given up, see above): it may
// take an eighth of the places that the stream's compute units have for it, so that eight such kernels of a like shape
// fit beside each other; kernels of any other kind end by themselves and make room.  A stream restricted to some
// compute units counts those only.
bool run_kernel_shape(int32_t n, int64_t d, int32_t B, bool vec, int32_t N, int64_t lda, hipStream_t st, RunShape* out) {
  const RunShape s = run_shape(n, d, B, vec);
  if (s.threads == 0 || lda >= (1LL << 30) / N) return false;    // an agent's rows within 32-bit distances: 4 GB
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if ((int64_t)n * s.nchunks * 8 > (int64_t)cus * s.wg_per_cu) return false;
  // (the handles of the legacy and the per-thread default stream are not pointers to a stream object, and nothing says
  // that the query takes them; like the null stream they carry no mask of their own)
  if (st == hipStreamLegacy || st == hipStreamPerThread) st = nullptr;
  uint32_t mask[32] = {};
  if (hipExtStreamGetCUMask(st, 32, mask) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  int usable = 0;
  for (uint32_t m : mask) usable += __builtin_popcount(m);
  const bool all_units = usable >= cus;
  if (!all_units) cus = usable;
  if ((int64_t)n * s.nchunks * 8 > (int64_t)cus * s.wg_per_cu) return false;
  *out = s;
  // Windows that need an eighth of one XCD's places (eight of a like shape fit there) play on one: n = 5, d = 1000, B = 8 1.92 ->
  // 1.68 us per iteration, n = 17, d = 180, B = 8 1.57 -> 1.38, n = 5, B = 32 3.2 -> 2.9.  Which one follows the workspace's
  // address, so that windows side by side spread.  Not on streams restricted to some compute units: that XCD may have too few of
  // them, and the window is then given up after its roll call.  Nor where the words of several agents share a line and many
  // workgroups of that XCD poll it: messages of one group (d = 4) gain 5 to 15 % up to 25 agents and lose up to 23 % from 35
  // on, other messages shorter than a line gain up to 45 and are even, 0.93 to 1.09 of the time, from 50 on.
  const int64_t message = run_row_words(s, d) * (int64_t)sizeof(unsigned long long);
  out->one_xcd = all_units && n <= (message == 32 ? 30 : message < 128 ? 48 : 64) && (int64_t)n * s.nchunks * 64 <= (int64_t)cus * s.wg_per_cu;
  return true;
}

template <int VEC, int THREADS, int BMAX, bool ODD, bool ONE_XCD>
static hipError_t launch(const RunArgs& a, hipStream_t st) {
  const int32_t kept = a.n * a.nchunks - g_tuning.window_missing;
  const unsigned wgs = (unsigned)(kept < 0 ? 0 : kept) + 1;                   // the last one calls the roll
  const dim3 grid(ONE_XCD ? wgs * 8 : wgs), block(THREADS);
  if (a.nchunks == 1) run_kernel<VEC, THREADS, BMAX, false, ODD, ONE_XCD><<<grid, block, 0, st>>>(a);
  else if constexpr (THREADS == 256 && VEC == 4) run_kernel<VEC, THREADS, BMAX, true, ODD, ONE_XCD><<<grid, block, 0, st>>>(a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_run(const RunArgs& a0, const RunShape& s, hipStream_t st) {
  RunArgs a = a0;
  a.dw = run_row_words(s, a.d);
  a.xcd = (int32_t)((reinterpret_cast<uintptr_t>(a.words) >> 12 ^ reinterpret_cast<uintptr_t>(a.words) >> 21) & 7);
  a.roll = a.words + run_kernel_words(s, a.n, a.d, a.B);
  const int64_t words = run_kernel_words(s, a.n, a.d, a.B) + 1;
  const int64_t blocks = (words + kBlock - 1) / kBlock;
  if (s.threads == 0 || a.B > s.bmax || a.nchunks != s.nchunks || a.tau < 1 || a.tau > kRunMaxTau || blocks > 0x7fffffffLL)
    return hipErrorInvalidValue;
  run_clear_kernel<<<dim3((unsigned)blocks), dim3(kBlock), 0, st>>>(a.words, words);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch ((s.vec ? 1 << 20 : 0) + s.threads * 64 + s.bmax - 1) {
#define CECA_RUN_XCD(VEC, T, BM, ODD) s.one_xcd ? launch<VEC, T, BM, ODD, true>(a, st) : launch<VEC, T, BM, ODD, false>(a, st)
#define CECA_RUN(VEC, T, BM) case (VEC == 4 ? 1 << 20 : 0) + T * 64 + BM - 1: if (VEC == 4 && a.d % 4) return CECA_RUN_XCD(VEC, T, BM, VEC == 4); return CECA_RUN_XCD(VEC, T, BM, false)
    CECA_RUN(4, 64, 8); CECA_RUN(4, 64, 16); CECA_RUN(4, 64, 32); CECA_RUN(4, 64, 64);
    CECA_RUN(4, 256, 8); CECA_RUN(4, 256, 16); CECA_RUN(4, 256, 32); CECA_RUN(4, 256, 64);
    CECA_RUN(4, 1024, 8); CECA_RUN(4, 1024, 16);
    CECA_RUN(1, 64, 16); CECA_RUN(1, 64, 64);
    CECA_RUN(1, 256, 16); CECA_RUN(1, 256, 64);
#undef CECA_RUN
#undef CECA_RUN_XCD
  }
  return hipErrorInvalidValue;
}

}  // namespace ceca
