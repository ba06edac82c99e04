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
// only on earlier ones: with every workgroup resident (the host's rule) every wait ends.  Should one not (workgroups
// kept off the device for kGiveUpTicks), it gives up: NaN takes the place of the missing values, and the call ends.
//
// What bounds it: the latency of the chain rows -> margins -> barrier -> coefficients -> message -> peer, once per
// iteration (an exchange between workgroups takes about 1.3 us), and a compute unit's intake of sampled rows, 75 GB/s.
// Per iteration, one launch (two in chunks) each before and here: n = 5, d = 1000, B = 8: 3.9 -> 1.9 us; n = 258, d = 10,
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

constexpr long long kGiveUpTicks = 30LL * 100 * 1000 * 1000;     // 30 s of the 100 MHz clock

__device__ __forceinline__ Word peek(const Word* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void publish(Word* p, uint32_t tag, float v) {
  __hip_atomic_store(p, ((Word)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A bounded wait: false once it has been given up, then for good.
struct Patience {
  bool lost = false;
  uint32_t polls = 0;
  long long since = 0;
  __device__ __forceinline__ void begin() { polls = 0; }
  __device__ __forceinline__ bool again() {
    if (lost) return false;
    if ((++polls & 1023u) == 0) {
      const long long now = wall_clock64();
      if (polls == 1024u) since = now;
      else if (now - since > kGiveUpTicks) { lost = true; return false; }
    }
    return true;
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
// columns and about 70 more registers per thread, nothing spilled
template <int VEC, int THREADS, int BMAX>
constexpr int run_waves() { return THREADS == 1024 || VEC == 1 || BMAX <= 8 ? 4 : BMAX <= 16 ? 3 : BMAX <= 32 ? 2 : 1; }

template <int VEC, int THREADS, int BMAX, bool CHUNKS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(run_waves<VEC, THREADS, BMAX>(), 8)))
void run_kernel(const RunArgs P) {
  using V = typename VecOf<VEC>::T;
  constexpr int WAVES = THREADS / 64;
  constexpr int CH = kRowGroup;            // rows are requested and added up in groups, as in the single-step kernels
  constexpr int MG = BMAX < 16 ? BMAX : 16;    // samples per wavefront sum (any number gives the same bits)
  static_assert(BMAX % CH == 0 && BMAX <= 64, "whole groups of samples, one lane per sample");
  __shared__ float red[2][WAVES][BMAX];    // alternating between iterations
  __shared__ float part[CHUNKS ? kRunParts : 1];                  // partial margins of every chunk of the agent
  const int agent = CHUNKS ? (int)(blockIdx.x / (uint32_t)P.nchunks) : (int)blockIdx.x;
  const int chunk = CHUNKS ? (int)(blockIdx.x % (uint32_t)P.nchunks) : 0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // lanes past the last column carry z = 0; they publish and wait for nothing
  const int64_t c = ((int64_t)chunk * THREADS + tid) * VEC;
  const bool on = c < P.d;
  const int64_t col = on ? c : 0;
  // message words of an agent: VEC planes of d / VEC words, so that neighbouring lanes touch neighbouring words
  const int64_t plane = P.d / VEC;
  const int64_t mine = (int64_t)agent * P.d + col / VEC;

  V x = ld_plain<V>(P.xin + (int64_t)agent * P.ld + col);
  V y = ld_plain<V>(P.yin + (int64_t)agent * P.ld + col);
  // a row's address is the agent's base in scalar registers plus 32 bits (the host sees to it that they are enough):
  // the row's distance, computed once per batch in lane j for sample j, and the thread's own offset
  const char* Abase = reinterpret_cast<const char*>(P.A + (int64_t)agent * P.N * P.lda + (int64_t)chunk * THREADS * VEC);
  const uint32_t voff = on ? (uint32_t)tid * VEC * 4 : 0;        // lanes past the last column read the chunk's first one
  const float* tbase = P.t + (int64_t)agent * P.N;
  const int32_t* idx = P.batch_idx + (int64_t)agent * P.B + min(lane, P.B - 1);    // samples past B repeat the last
  const int64_t nb = (int64_t)P.n * P.B;
  int32_t myidx = min(max(idx[0], 0), P.N - 1);
  V a[BMAX];
#pragma unroll
  for (int j = 0; j < BMAX; ++j) a[j] = V(0.0f);      // groups past B are never requested
  float tmine;
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
  int32_t idx_next = idx[P.iters > 1 ? nb : 0];
  Patience wait;
  int r = P.r0;
  int reader = agent;                      // who read my message two iterations ago (after the shifts below)
  int reader1 = agent;                     // and one iteration ago
  for (int t = 0; t < P.iters; ++t) {
    const int par = t & 1;
    const MultiRound& R = P.round[r];
    const uint32_t tag = (uint32_t)t + 1;
    // the look at the reader of my message of iteration t - 2: has it published iteration t - 1?
    const Word* seen = P.words + (int64_t)(par ^ 1) * P.n * P.d + (int64_t)reader * P.d + col / VEC;
    Word ack = 0;
    if (t >= 2 && on) ack = peek(seen);

    const V z = on ? (R.exch_y ? y : x) : V(0.0f);
    // every group of the tile, also those past B (zeros): without branches the groups' chains overlap
#pragma unroll
    for (int c0 = 0; c0 < BMAX; c0 += MG) {
      float m[MG];
#pragma unroll
      for (int j = 0; j < MG; ++j) m[j] = dot_v(a[c0 + j], z);
      int jrow;
      bool owner;
      const float msum = wave_sum_many<MG>(m, lane, jrow, owner);
      if (owner) red[par][wave][c0 + jrow] = msum;
    }
    __syncthreads();
    float mj = 0.0f;
    if (CHUNKS) {
      Word* ring = P.words + 2 * (int64_t)P.n * P.d + ((int64_t)par * P.n + agent) * P.nchunks * P.B;
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
        part[i0] = (uint32_t)(w0 >> 32) == tag ? __uint_as_float((uint32_t)w0) : __builtin_nanf("");
        part[i1] = (uint32_t)(w1 >> 32) == tag ? __uint_as_float((uint32_t)w1) : __builtin_nanf("");
      }
      __syncthreads();
      const int j = min(lane, P.B - 1);
      for (int ch = 0; ch < P.nchunks; ++ch) mj += part[ch * P.B + j];
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
    if (P.noise_std != 0.0f) e = add_noise<V>(e, P.noise_std, col, noise_keys(P.seed, P.k + (uint32_t)t, (uint32_t)agent));
    const V v = z - P.lr * e;

    int p, to;                             // whose message I read, and who reads mine (Eqs. (6), (7))
    if (P.port == 2) {
      p = agent - R.shift; if (p < 0) p += P.n;
      to = agent + R.shift; if (to >= P.n) to -= P.n;
    } else {
      p = (agent & 1) ? agent - R.shift : agent + R.shift;
      if (p < 0) p += P.n;
      if (p >= P.n) p -= P.n;
      to = p;
    }
    if (t >= 2 && on) {
      wait.begin();
      while ((uint32_t)(ack >> 32) < (uint32_t)t && wait.again()) ack = peek(seen);
    }
    if (on) {
      Word* slot = P.words + (int64_t)par * P.n * P.d + mine;
#pragma unroll
      for (int u = 0; u < VEC; ++u) publish(slot + u * plane, tag, Parts<VEC>::get(v, u));
    }
    // the next iteration's rows travel while the message does; a batch of the same rows (full gradients) is there
    if (t + 1 < P.iters) {
      const int32_t now = myidx;
      myidx = min(max(idx_next, 0), P.N - 1);
      if (__any(now != myidx)) request_rows();                   // the same in every wavefront
      idx_next = idx[(int64_t)min(t + 2, P.iters - 1) * nb];
    }
    V msg = V(0.0f);
    if (on) {
      const Word* slot = P.words + (int64_t)par * P.n * P.d + (int64_t)p * P.d + col / VEC;
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
        Parts<VEC>::set(msg, u, (uint32_t)(w[u] >> 32) == tag ? __uint_as_float((uint32_t)w[u]) : __builtin_nanf(""));
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
  if (on) {
    *reinterpret_cast<V*>(P.xout + (int64_t)agent * P.ld + col) = x;
    *reinterpret_cast<V*>(P.yout + (int64_t)agent * P.ld + col) = y;
  }
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
  RunShape s{0, 0, 1, 0};
  if (n < 2 || B < 1 || B > 64) return s;
  const int64_t groups = vec4 ? d / 4 : d;
  if (vec4) {
    if (groups <= 64) s.threads = 64;                            // (the single step's other wavefronts add zeros)
    else if (groups <= 256) s.threads = 256;
    else if (groups <= 1024 && B <= 16) s.threads = 1024;
    else if (grad_fused_covers(n, d, B, true)) return s;         // wider rows in one workgroup
    else s.threads = 256;
  } else {
    s.threads = groups <= 64 ? 64 : groups <= 256 ? 256 : groups <= 1024 ? 1024 : 256;
  }
  const int64_t chunks = (groups + s.threads - 1) / s.threads;
  if (chunks * B > kRunParts && chunks > 1) return RunShape{0, 0, 1, 0};
  s.nchunks = (int32_t)chunks;
  s.bmax = vec4 ? (B <= 8 ? 8 : B <= 16 ? 16 : B <= 32 ? 32 : 64) : (B <= 16 ? 16 : 64);
  const int waves = s.threads == 1024 || !vec4 || s.bmax <= 8 ? 4 : s.bmax <= 16 ? 3 : s.bmax <= 32 ? 2 : 1;     // run_waves
  s.wg_per_cu = 4 * waves / (s.threads / 64);
  return s;
}

int64_t run_kernel_words(const RunShape& s, int32_t n, int64_t d, int32_t B) {
  return 2 * (int64_t)n * d + (s.nchunks > 1 ? 2 * (int64_t)n * s.nchunks * B : 0);
}

// Every workgroup of the kernel has to be resident, whatever else runs: it may take an eighth of the places that the
// stream's compute units have for it, so that eight such kernels fit beside each other (a process has four
// hardware queues); kernels of any other kind end by themselves and make room.  A stream restricted to some compute
// units counts those only.
bool run_kernel_shape(int32_t n, int64_t d, int32_t B, int32_t N, int64_t lda, bool vec4, hipStream_t st, RunShape* out) {
  const RunShape s = run_shape(n, d, B, vec4);
  if (s.threads == 0 || lda >= (1LL << 30) / N) return false;    // an agent's rows within 32-bit distances: 4 GB
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if ((int64_t)n * s.nchunks * 8 > (int64_t)cus * s.wg_per_cu) return false;
  uint32_t mask[32] = {};
  if (hipExtStreamGetCUMask(st, 32, mask) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  int usable = 0;
  for (uint32_t m : mask) usable += __builtin_popcount(m);
  if (usable < cus) cus = usable;
  if ((int64_t)n * s.nchunks * 8 > (int64_t)cus * s.wg_per_cu) return false;
  *out = s;
  return true;
}

template <int VEC, int THREADS, int BMAX>
static hipError_t launch(const RunArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)(a.n * a.nchunks)), block(THREADS);
  if (a.nchunks == 1) run_kernel<VEC, THREADS, BMAX, false><<<grid, block, 0, st>>>(a);
  else if constexpr (THREADS == 256) run_kernel<VEC, THREADS, BMAX, true><<<grid, block, 0, st>>>(a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_run(const RunArgs& a, const RunShape& s, bool vec4, hipStream_t st) {
  const int64_t words = run_kernel_words(s, a.n, a.d, a.B);
  const int64_t blocks = (words + kBlock - 1) / kBlock;
  if (s.threads == 0 || a.B > s.bmax || a.nchunks != s.nchunks || a.tau < 1 || a.tau > kRunMaxTau || blocks > 0x7fffffffLL)
    return hipErrorInvalidValue;
  run_clear_kernel<<<dim3((unsigned)blocks), dim3(kBlock), 0, st>>>(a.words, words);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch ((vec4 ? 1 << 20 : 0) + s.threads * 64 + s.bmax - 1) {
#define CECA_RUN(VEC, T, BM) case (VEC == 4 ? 1 << 20 : 0) + T * 64 + BM - 1: return launch<VEC, T, BM>(a, st)
    CECA_RUN(4, 64, 8); CECA_RUN(4, 64, 16); CECA_RUN(4, 64, 32); CECA_RUN(4, 64, 64);
    CECA_RUN(4, 256, 8); CECA_RUN(4, 256, 16); CECA_RUN(4, 256, 32); CECA_RUN(4, 256, 64);
    CECA_RUN(4, 1024, 8); CECA_RUN(4, 1024, 16);
    CECA_RUN(1, 64, 16); CECA_RUN(1, 64, 64);
    CECA_RUN(1, 256, 16); CECA_RUN(1, 256, 64);
    CECA_RUN(1, 1024, 16); CECA_RUN(1, 1024, 64);
#undef CECA_RUN
  }
  return hipErrorInvalidValue;
}

}  // namespace ceca
