// Branch Speculative Sampling at one node, and the accept/resample walk over
// a token tree (Preliminaries, "Speculative Decoding"; Appendix, Algorithm 1
// "Branch Speculative Sampling"):
//   p(v)   = fl32(exp(fl32(fl32(l_v * fl32(1/T)) - zmax))) / total  (float64)
//            or the one-hot at argmax when T = 0;
//   accept = float64(u) < p~(x) / float64(q(x));
//   reject : p~ <- max(0, p~ - q) / Z,  Z = sum max(0, p~ - q)   (float64),
//            Z <= 0 keeps p~ and raises SB_FLAG_ZERO_RESIDUAL;
//   draw   : C_v = running float64 sum of p~ in vocabulary order,
//            y = min{v : C_v > u * W}, W the float64 total; a zero-mass
//            token is never drawn.
// The multiply-then-subtract of the logit transform must not be contracted
// into an FMA: every operation rounds on its own, as the definition states.
//
// A walk is a chain of dependent vocabulary passes (each residual needs the
// mass of the one before), so one compute unit's path to memory bounds it
// when one workgroup does the passes: 12 us a pass at 32000 tokens, 30 at
// 128256.  Here G workgroups of 256 threads share the vocabulary, 1024 to
// 8192 consecutive tokens each, and keep their slice of p~ in registers from
// pass to pass (nothing but q is read again).  All of them take the same
// decisions from the same values; after a rejection each publishes its
// slice's mass and the residual at the next candidate's token, and reads
// everyone else's.  A draw looks up the slice masses it already has; only the
// workgroup of the crossing slice searches its tokens, and sends the one it
// finds to workgroup 0, which alone writes the result: when any message it
// needs stays out (a workgroup that gave up, or that the chip has no room for)
// it does the walk again by itself with p~ in memory.  Measured (the walk
// and the launch that clears the messages, in turn on an idle device; one
// workgroup of 1024 threads -> these): a chain rejected at its first draft, 32000
// tokens 20 -> 13 us, 128256 tokens 54 -> 14; a chain accepted whole 14 -> 12 and
// 29 -> 13; a selection with three rejections 45 -> 19 and 156 -> 21, one accepted
// at once 8 -> 10 to 12 (the clearing launch: 4.6 us in a kernel trace, of which
// 2 to 3 show).  The token's way to workgroup 0 is about 1 us of these.
#pragma clang fp contract(off)

#include <limits.h>
#include <math.h>

#include "sb_device.h"
#include "sb_internal.h"

namespace sb {
namespace {

constexpr int kT = 256;      // threads of a workgroup
constexpr int kMemT = 1024;  // of the one past the slices' reach
constexpr int kMaxG = 256;  // workgroups: one thread per slice mass
__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Inclusive 64-lane scan.
__device__ __forceinline__ double wave_scan(double x) {
  const int lane = threadIdx.x & 63;
  for (int o = 1; o < 64; o <<= 1) {
    const double y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

// A target row's distribution; raw(v) is p before the factor scale().
struct Row {
  float inv_t, zmax;
  double total;
  int argmax, greedy;
  __device__ __forceinline__ double raw(float l, int v) const {
    if (greedy) return v == argmax ? 1.0 : 0.0;
    const float z = l * inv_t;
    return (double)expf(z - zmax);
  }
  __device__ __forceinline__ double scale() const { return greedy ? 1.0 : 1.0 / total; }
  // p(v) divided exactly (the accept ratio of a tested token)
  __device__ __forceinline__ double at(float l, int v) const {
    if (greedy) return v == argmax ? 1.0 : 0.0;
    const float z = l * inv_t;
    return (double)expf(z - zmax) / total;
  }
};

struct WalkShared {
  double part[kMemT / 64], part2[kMemT / 64];
  double z, cap;
  int fail, first, last;
  int32_t token;  // the draw's
};

// Messages between the workgroups.  Word 0 is the drawn token + 1 (0: not there
// yet), sent to workgroup 0.  Then per exchange and workgroup two words, the
// complement of a float64's bits (a NaN as the canonical one), never 0; 0 is
// "not there yet".  Three sets take turns: exchange k uses set k % 3, and its
// publisher first clears its words of set (k + 1) % 3 -- they held exchange
// k - 2, which everyone has read, since everyone published k - 1 after it --
// and waits for that store, so who sees message k sees the cleared words.  Only
// word 0 and the first set are clear before the launch.
// Words move with device-scope relaxed stores and loads; the message is the
// data, nothing else crosses workgroups.
__device__ __forceinline__ unsigned long long encode(double v) {
  if (v != v) return ~0x7ff8000000000000ull;
  return ~__builtin_bit_cast(unsigned long long, v);
}
__device__ __forceinline__ double decode(unsigned long long w) {
  return __builtin_bit_cast(double, ~w);
}
__device__ __forceinline__ void put(unsigned long long *p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long get(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Block-wide sums of v and c (every thread gets them).
template <int NT>
__device__ void block_sum2(double &v, double &c, WalkShared &sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  v = wave_sum(v);
  c = wave_sum(c);
  if (lane == 0) {
    sh.part[w] = v;
    sh.part2[w] = c;
  }
  __syncthreads();
  v = c = 0.0;
#pragma unroll
  for (int k = 0; k < NT / 64; k += 4) {
    v += (sh.part[k] + sh.part[k + 1]) + (sh.part[k + 2] + sh.part[k + 3]);
    c += (sh.part2[k] + sh.part2[k + 1]) + (sh.part2[k + 2] + sh.part2[k + 3]);
  }
  __syncthreads();
}

// Block-wide inclusive scan of v in thread order.
__device__ double block_scan(double v, WalkShared &sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double inc = wave_scan(v);
  if (lane == 63) sh.part[w] = inc;
  __syncthreads();
  double off = 0.0;
  for (int k = 0; k < w; ++k) off += sh.part[k];
  __syncthreads();
  return off + inc;
}

// The first thread whose inclusive sum inc passes thr with mass of its own;
// when rounding leaves none, the last thread with mass; -1 without any mass.
__device__ int block_cross(double mass, double inc, double thr, WalkShared &sh) {
  if (threadIdx.x == 0) {
    sh.first = INT_MAX;
    sh.last = -1;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const unsigned long long hit = __ballot(mass > 0.0 && inc > thr), any = __ballot(mass > 0.0);
  if (lane == 0) {
    const int base = threadIdx.x;
    if (hit) atomicMin(&sh.first, base + __ffsll((long long)hit) - 1);
    if (any) atomicMax(&sh.last, base + 63 - __clzll((long long)any));
  }
  __syncthreads();
  const int r = sh.first != INT_MAX ? sh.first : sh.last;
  __syncthreads();
  return r;
}

// The current distribution p~ = x scale of this workgroup's EPT kT tokens in
// registers, thread t the EPT consecutive ones from v0.
template <int EPT>
struct Slices {
  static constexpr int kThreads = kT;
  int vocab, vec4, G, g, v0;
  unsigned long long *msg;  // 1 + [3][G][2]
  int k;                    // exchanges so far
  WalkWait wait;
  double x[EPT], scale, zdiv;
  double mass;  // of workgroup threadIdx.x's slice, once have_mass
  bool have_mass;

  __device__ void init(int vocab_, int vec4_, const WalkWait &wait_, unsigned long long *msg_) {
    vocab = vocab_;
    vec4 = vec4_;
    G = gridDim.x;
    g = blockIdx.x;
    v0 = (g * kT + (int)threadIdx.x) * EPT;
    msg = msg_;
    k = 0;
    wait = wait_;
  }
  // This workgroup does not wait now (a test's).
  __device__ __forceinline__ bool gives_up() const { return g >= wait.lo && g < wait.hi && k >= wait.at; }
  __device__ __forceinline__ void load(const float *row, float (&f)[EPT]) const {
    const __amdgpu_buffer_rsrc_t rs = uniform_rsrc(row, vocab * 4);
    if (vec4) {
#pragma unroll
      for (int e = 0; e < EPT; e += 4) {
        const f32x4 t = __builtin_bit_cast(
            f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (v0 + e) * 4, 0, 0));
        f[e] = t[0];
        f[e + 1] = t[1];
        f[e + 2] = t[2];
        f[e + 3] = t[3];
      }
    } else {
#pragma unroll
      for (int e = 0; e < EPT; ++e)
        f[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (v0 + e) * 4, 0, 0));
    }
  }
  __device__ void set_row(const Row &r, const float *l) {
    float f[EPT];
    load(l, f);
#pragma unroll
    for (int e = 0; e < EPT; ++e) x[e] = v0 + e < vocab ? r.raw(f[e], v0 + e) : 0.0;
    scale = r.scale();
    have_mass = false;
  }
  // Publishes this slice's sum and cap (only the thread that has one passes a
  // cap) and reads everyone's: sh.z = the sum of the sums, sh.cap = the cap,
  // own = workgroup threadIdx.x's sum.  False when a message stays out.
  __device__ bool exchange(double sum, double cap, double &own, WalkShared &sh) {
    block_sum2<kT>(sum, cap, sh);
    if (threadIdx.x == 0) sh.fail = 0;
    double s = threadIdx.x == 0 ? sum : 0.0, c = threadIdx.x == 0 ? cap : 0.0;
    if (G > 1) {
      unsigned long long *cur = msg + 1 + (size_t)(k % 3) * G * 2;
      unsigned long long *nxt = msg + 1 + (size_t)((k + 1) % 3) * G * 2;
      const bool leave = gives_up();
      ++k;
      if (threadIdx.x == 0) {
        put(nxt + 2 * g, 0ull);
        put(nxt + 2 * g + 1, 0ull);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        put(cur + 2 * g, encode(sum));
        put(cur + 2 * g + 1, encode(cap));
      }
      __syncthreads();
      s = c = 0.0;
      if ((int)threadIdx.x < G) {
        const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
        unsigned long long x = 0, y = 0;
        for (;;) {
          if (!x) x = get(cur + 2 * threadIdx.x);
          if (!y) y = get(cur + 2 * threadIdx.x + 1);
          if (x && y && !leave) break;
          if (leave || __builtin_amdgcn_s_memrealtime() - t0 > wait.ticks) {
            sh.fail = 1;
            break;
          }
        }
        s = x ? decode(x) : 0.0;
        c = y ? decode(y) : 0.0;
      }
    }
    own = s;
    block_sum2<kT>(s, c, sh);
    if (threadIdx.x == 0) {
      sh.z = s;
      sh.cap = c;
    }
    __syncthreads();
    return sh.fail == 0;
  }
  // p~ <- max(0, p~ - q) / Z when Z > 0; sh.z = Z, sh.cap = the residual at
  // token xcap (when xcap >= 0).
  __device__ bool reject(const float *q, int xcap, WalkShared &sh) {
    float f[EPT];
    load(q, f);
    double r[EPT], part = 0.0, cap = 0.0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      r[e] = x[e] * scale - (double)f[e];
      r[e] = r[e] > 0.0 && v0 + e < vocab ? r[e] : 0.0;
      part += r[e];
      cap = v0 + e == xcap ? r[e] : cap;
    }
    double own;
    if (!exchange(part, cap, own, sh)) return false;
    if (sh.z > 0.0) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) x[e] = r[e];
      zdiv = sh.z;
      scale = 1.0 / zdiv;
      mass = own;
      have_mass = true;
    }
    return true;
  }
  // sh.cap = the residual at token v.
  __device__ bool fetch(int v, WalkShared &sh) {
    double cap = 0.0, own;
#pragma unroll
    for (int e = 0; e < EPT; ++e) cap = v0 + e == v ? x[e] : cap;
    return exchange(0.0, cap, own, sh);
  }
  // In workgroup 0 sh.token is the token; false there when it stays out.
  __device__ bool draw(float u, WalkShared &sh) {
    double ts = 0.0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) ts += x[e];
    if (!have_mass && !exchange(ts, 0.0, mass, sh)) return false;
    const double m = mass, inc = block_scan(m, sh);
    if ((int)threadIdx.x == kT - 1) sh.z = inc;  // W: slices past G have none
    __syncthreads();
    const double thr = (double)u * sh.z;
    const int cross = block_cross(m, inc, thr, sh);
    if (cross < 0) {
      if (threadIdx.x == 0) sh.token = vocab - 1;
      return true;
    }
    if (cross == g) {
      if ((int)threadIdx.x == cross) sh.cap = inc - m;
      __syncthreads();
      const double base = sh.cap, tinc = base + block_scan(ts, sh);
      const int at = block_cross(ts, tinc, thr, sh);
      if ((int)threadIdx.x == (at < 0 ? 0 : at)) {
        int found = -1, last = v0;
        double c = tinc - ts;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
          c += x[e];
          if (x[e] > 0.0) {
            last = v0 + e;
            if (found < 0 && c > thr) found = v0 + e;
          }
        }
        sh.token = found >= 0 ? found : last;
        if (g != 0) put(msg, (unsigned long long)sh.token + 1);
      }
      return true;
    }
    if (g != 0) return true;
    if (threadIdx.x == 0) {
      const bool leave = gives_up();
      const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
      unsigned long long w;
      sh.fail = 0;
      for (;;) {
        w = get(msg);
        if (w && !leave) break;
        if (leave || __builtin_amdgcn_s_memrealtime() - t0 > wait.ticks) {
          sh.fail = 1;
          break;
        }
      }
      sh.token = (int32_t)w - 1;
    }
    __syncthreads();
    return sh.fail == 0;
  }
};

// The same by one workgroup of NT threads with p~ in memory: after a message
// stayed out, and for vocabularies past the slices' reach.  Bound by one compute
// unit's path to memory, so every pass reads along the vocabulary, kBatch loads
// of a thread in flight.  Three rejections and a draw at 2100001 tokens: 2.1 ms
// (24 with a stretch of the vocabulary per thread); 256 threads after a give-up:
// 79 us at 32000 tokens (205), 257 at 128256 (775).
template <int NT>
struct InMemory {
  static constexpr int kThreads = NT, kBatch = 16;
  // arr holds a residual r where r > 0 and elsewhere minus the p~ it was taken
  // from, so a residual without mass, minus p~ everywhere, still has p~.
  enum { kRow, kResidual, kKept };
  int vocab, state;
  double *arr;
  Row row;
  const float *l;
  double scale, zdiv;
  __device__ __forceinline__ void set_row(const Row &r, const float *lrow) {
    row = r;
    l = lrow;
    scale = r.scale();
    state = kRow;
  }
  // p~ / scale at the tokens v (outside [0, hi): 0).
  template <int K>
  __device__ __forceinline__ void load(const int (&v)[K], int hi, double (&x)[K]) const {
    if (state == kRow) {
      const __amdgpu_buffer_rsrc_t rs = uniform_rsrc(l, vocab * 4);
      float f[K];
#pragma unroll
      for (int k = 0; k < K; ++k)
        f[k] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(rs, (v[k] < hi ? v[k] : vocab) * 4, 0, 0));
#pragma unroll
      for (int k = 0; k < K; ++k) x[k] = v[k] < hi ? row.raw(f[k], v[k]) : 0.0;
    } else {
      const __amdgpu_buffer_rsrc_t rs = uniform_rsrc(arr, vocab * 8);
#pragma unroll
      for (int k = 0; k < K; ++k)
        x[k] = __builtin_bit_cast(
            double, __builtin_amdgcn_raw_buffer_load_b64(rs, (v[k] < hi ? v[k] : vocab) * 8, 0, 0));
#pragma unroll
      for (int k = 0; k < K; ++k) x[k] = state == kKept ? -x[k] : x[k] > 0.0 ? x[k] : 0.0;
    }
  }
  __device__ __forceinline__ void load_run(int v0, int hi, double (&x)[kBatch]) const {
    int v[kBatch];
#pragma unroll
    for (int b = 0; b < kBatch; ++b) v[b] = v0 + b;
    load(v, hi, x);
  }
  __device__ __forceinline__ bool reject(const float *q, int xcap, WalkShared &sh) {
    if (threadIdx.x == 0) sh.cap = 0.0;
    __syncthreads();
    const __amdgpu_buffer_rsrc_t qrs = uniform_rsrc(q, vocab * 4);
    double part = 0.0, none = 0.0;
    for (int v0 = threadIdx.x; v0 < vocab; v0 += kBatch * NT) {
      int v[kBatch];
      float qv[kBatch];
      double x[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        v[b] = v0 + b * NT;
        qv[b] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(qrs, (v[b] < vocab ? v[b] : vocab) * 4, 0, 0));
      }
      load(v, vocab, x);
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const double r = x[b] * scale - (double)qv[b];
        if (v[b] < vocab) {
          arr[v[b]] = r > 0.0 ? r : -x[b];
          part += r > 0.0 ? r : 0.0;
          if (v[b] == xcap) sh.cap = r > 0.0 ? r : 0.0;
        }
      }
    }
    block_sum2<NT>(part, none, sh);
    if (threadIdx.x == 0) sh.z = part;
    if (part > 0.0) {
      zdiv = part;
      scale = 1.0 / zdiv;
      state = kResidual;
    } else if (state != kRow) {
      state = kKept;
    }
    __syncthreads();
    return true;
  }
  __device__ __forceinline__ bool fetch(int v, WalkShared &sh) {
    const int at[1] = {v};
    double x[1];
    load(at, vocab, x);
    if (threadIdx.x == 0) sh.cap = x[0];
    __syncthreads();
    return true;
  }
  // The wave whose stretch of the vocabulary crosses, then the thread whose run
  // of that stretch does, then the token.
  __device__ __forceinline__ bool draw(float u, WalkShared &sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int per = (vocab + NT / 64 - 1) / (NT / 64);
    double mass = 0.0;
    for (int v0 = w * per + lane; v0 < min(vocab, (w + 1) * per); v0 += kBatch * 64) {
      int v[kBatch];
      double x[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) v[b] = v0 + b * 64;
      load(v, min(vocab, (w + 1) * per), x);
#pragma unroll
      for (int b = 0; b < kBatch; ++b) mass += x[b];
    }
    mass = wave_sum(mass);
    if (lane != 0) mass = 0.0;
    const double inc = block_scan(mass, sh);
    if ((int)threadIdx.x == NT - 1) sh.z = inc;
    __syncthreads();
    const double thr = (double)u * sh.z;
    const int cross = block_cross(mass, inc, thr, sh);
    if (cross < 0) {
      if (threadIdx.x == 0) sh.token = vocab - 1;
      __syncthreads();
      return true;
    }
    if ((int)threadIdx.x == cross) sh.cap = inc - mass;
    __syncthreads();
    const double base = sh.cap;
    const int end = min(vocab, ((cross >> 6) + 1) * per), run = (per + NT - 1) / NT;
    const int lo = (cross >> 6) * per + (int)threadIdx.x * run, hi = min(end, lo + run);
    double ts = 0.0;
    for (int v0 = lo; v0 < hi; v0 += kBatch) {
      double x[kBatch];
      load_run(v0, hi, x);
#pragma unroll
      for (int b = 0; b < kBatch; ++b) ts += x[b];
    }
    const double tinc = base + block_scan(ts, sh);
    const int at = block_cross(ts, tinc, thr, sh);
    if ((int)threadIdx.x == (at < 0 ? 0 : at)) {
      int found = -1, last = lo;
      double c = tinc - ts;
      for (int v0 = lo; v0 < hi; v0 += kBatch) {
        double x[kBatch];
        load_run(v0, hi, x);
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
          c += x[b];
          if (x[b] > 0.0) {
            last = v0 + b;
            if (found < 0 && c > thr) found = v0 + b;
          }
        }
      }
      sh.token = found >= 0 ? found : last;
    }
    __syncthreads();
    return true;
  }
};

// One call: the tree (select: a root with n - 1 children, row i of q and u
// being candidate i - 1's) and its rows' values, in LDS.
constexpr int kRows = SB_MAX_ROWS + 1;
struct WalkRows {
  int n;
  int16_t par[kRows], path[kRows], kids[kRows];
  int32_t tok[kRows], first[kRows];  // first: lowest-index child (INT_MAX: none)
  float u[kRows], qx[kRows];         // qx: q of the row at its token
  double px[kRows];                  // p of the row's parent at the row's token
  sb_row_stats st[kRows];
  unsigned long long kmask[kMemT / 64];
  int node, plen, nk, decision, flags;
};
static_assert(SB_MAX_ROWS <= kT, "a walk's rows have a thread each");

struct WalkIn {
  int vocab, n, greedy;
  float inv_t;
  const int32_t *tokens;  // of row i: tokens[i - off]
  const float *logits;
  const sb_row_stats *stats;
  const float *q, *u;  // rows i - off
  int off;             // 0: walk; 1: select
  int u_draw;          // index of the final draw's uniform
};

// A row whose total is not finite (a NaN or +inf logit, an invalid forward) has
// no mass at T > 0: its every raw(v) is NaN.
__device__ __forceinline__ Row row_of(const WalkIn &a, const sb_row_stats &s) {
  return Row{a.inv_t, isfinite(s.total) ? s.zmax : NAN, s.total, s.argmax, a.greedy};
}

// The accept test of row c against p~(its token) = px (thread 0).
__device__ __forceinline__ bool accept(const WalkIn &a, const WalkRows &R, int c, double px, int *flags) {
  const int x = R.tok[c];
  double ratio = 0.0;  // a token id outside the vocabulary is rejected
  if (x >= 0 && x < a.vocab) {
    const double qx = (double)R.qx[c];
    if (qx == 0.0) *flags |= SB_FLAG_QZERO;
    ratio = px / qx;
  } else {
    *flags |= SB_FLAG_QZERO;
  }
  return (double)R.u[c] < ratio;
}

// The walk from the root.  Returns false when a message stayed out; else sh.token
// is workgroup 0's drawn token (`select`: only without an acceptance), *bonus
// whether a leaf was reached.
template <class D>
__device__ bool walk_run(D &d, const WalkIn &a, WalkRows &R, WalkShared &sh, bool select, int *nrej,
                         int *bonus) {
  constexpr int NT = D::kThreads;
  for (;;) {
    // While a node's first candidate is accepted against the node's own row,
    // the tests read LDS only, and one thread walks them.  The failing one is
    // taken again below, with its rejection.
    if (threadIdx.x == 0 && !select) {
      for (;;) {
        const int c = R.first[R.node];
        if (c == INT_MAX || !accept(a, R, c, R.px[c], &R.flags)) break;
        R.path[R.plen++] = (int16_t)c;
        R.node = c;
      }
    }
    __syncthreads();
    const int node = R.node;
    // the children of `node` in index order, one thread per row (a selection's
    // are all the other rows)
    if (select) {
      for (int j = threadIdx.x + 1; j < a.n; j += NT) R.kids[j - 1] = (int16_t)j;
      if (threadIdx.x == 0) R.nk = a.n - 1;
    } else {
      const int j = threadIdx.x, w = j >> 6;
      const unsigned long long m = __ballot(j > node && j < a.n && R.par[j] == node);
      if ((j & 63) == 0) R.kmask[w] = m;
      __syncthreads();
      int before = __popcll(m & ((1ull << (j & 63)) - 1));
      for (int v = 0; v < w; ++v) before += __popcll(R.kmask[v]);
      if ((m >> (j & 63)) & 1) R.kids[before] = (int16_t)j;
      if (j == NT - 1) R.nk = before + (int)((m >> 63) & 1);
    }
    __syncthreads();
    const int nk = R.nk;
    d.set_row(row_of(a, R.st[node]), a.logits + (size_t)node * a.vocab);
    *bonus = nk == 0;
    int acc = -1;
    bool resid = false;  // p~ is a residual
    double px_at = 0.0;  // p~ at the next candidate's token, once it is
    for (int i = 0; i < nk; ++i) {
      const int c = R.kids[i];
      if (threadIdx.x == 0) R.decision = accept(a, R, c, resid ? px_at : R.px[c], &R.flags);
      __syncthreads();
      const int ok = R.decision;
      __syncthreads();
      if (ok) {
        acc = c;
        break;
      }
      ++*nrej;
      const int xn = i + 1 < nk ? R.tok[R.kids[i + 1]] : -1;
      const int xcap = xn >= 0 && xn < a.vocab ? xn : -1;
      if (!d.reject(a.q + (size_t)(c - a.off) * a.vocab, xcap, sh)) return false;
      const double Z = sh.z;
      if (Z > 0.0) {
        resid = true;
        px_at = sh.cap / Z;
      } else {
        if (threadIdx.x == 0) R.flags |= SB_FLAG_ZERO_RESIDUAL;
        if (resid && xcap >= 0) {
          __syncthreads();
          if (!d.fetch(xcap, sh)) return false;
          px_at = sh.cap / d.zdiv;
        }
      }
      __syncthreads();
    }
    if (acc < 0) return d.draw(a.u[a.u_draw], sh);
    if (threadIdx.x == 0) {
      R.path[R.plen++] = (int16_t)acc;
      R.node = acc;
    }
    if (select) return true;
    __syncthreads();
  }
}

// The rows' values, before the first test.
template <int NT>
__device__ void walk_rows(const WalkIn &a, const TreeArg *tree, WalkRows &R) {
  const int n = a.n;
  for (int i = threadIdx.x; i < n; i += NT) {
    R.par[i] = tree ? tree->parent[i] : (int16_t)(i == 0 ? -1 : 0);
    if (tree || i == 0) R.st[i] = a.stats[i];
    R.tok[i] = i >= a.off ? a.tokens[i - a.off] : -1;
    R.u[i] = i >= a.off ? a.u[i - a.off] : 0.0f;
    R.first[i] = INT_MAX;
  }
  if (threadIdx.x == 0) R.flags = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += NT) {
    if ((tree || i == 0) && isnan(R.st[i].total)) atomicOr(&R.flags, SB_FLAG_NONFINITE);
    if (i == 0) continue;
    const int par = R.par[i], x = R.tok[i];
    atomicMin(&R.first[par], i);
    double px = 0.0;
    float qx = 0.0f;
    if (x >= 0 && x < a.vocab) {
      px = row_of(a, R.st[par]).at(a.logits[(size_t)par * a.vocab + x], x);
      qx = a.q[(size_t)(i - a.off) * a.vocab + x];
    }
    R.px[i] = px;
    R.qx[i] = qx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    R.path[0] = 0;
    R.node = 0;
    R.plen = 1;
  }
  __syncthreads();
}

// EPT tokens per thread (0: one workgroup, p~ in memory).
template <int EPT, bool SELECT>
__global__ __launch_bounds__(EPT ? kT : kMemT) void k_walk(WalkIn a, TreeArg tree, int vec4, WalkWait wait,
                                             sb_step_result *__restrict__ result,
                                             int32_t *__restrict__ out,
                                             unsigned long long *msg, double *arr) {
  constexpr int NT = EPT ? kT : kMemT;
  __shared__ WalkRows R;
  __shared__ WalkShared sh;
  walk_rows<NT>(a, SELECT ? nullptr : &tree, R);
  int nrej = 0, bonus = 0;
  bool done = false;
  if constexpr (EPT > 0) {
    Slices<EPT> d;
    d.init(a.vocab, vec4, wait, msg);
    done = walk_run(d, a, R, sh, SELECT, &nrej, &bonus);
  }
  if (blockIdx.x != 0) return;  // the result is workgroup 0's alone
  if (!done) {
    if (EPT > 0) walk_rows<NT>(a, SELECT ? nullptr : &tree, R);
    nrej = bonus = 0;
    InMemory<NT> d;
    d.vocab = a.vocab;
    d.arr = arr;
    walk_run(d, a, R, sh, SELECT, &nrej, &bonus);
  }
  __syncthreads();
  if constexpr (SELECT) {
    if (threadIdx.x == 0) {
      const int acc = R.plen > 1 ? R.path[1] - 1 : -1;
      out[0] = acc;
      out[1] = acc >= 0 ? R.tok[acc + 1] : sh.token;
      out[2] = R.flags;
    }
  } else {
    if (threadIdx.x == 0) {
      int branch = -1;
      if (R.plen > 1) {
        branch = 0;
        for (int j = 1; j < R.path[1]; ++j)
          if (R.par[j] == 0) ++branch;
      }
      result->n_accepted = R.plen - 1;
      result->branch = branch;
      result->next_token = sh.token;
      result->path_len = R.plen;
      result->flags = R.flags;
      result->n_rejected = nrej;
      result->bonus = bonus;
      result->reserved = 0;
    }
    for (int j = threadIdx.x; j < SB_MAX_ROWS; j += NT)
      result->path[j] = j < R.plen ? (int32_t)R.path[j] : -1;
  }
}

__global__ __launch_bounds__(kT) void k_walk_clear(unsigned long long *p, int n) {
  for (int i = threadIdx.x; i < n; i += kT) p[i] = 0;
}

// One workgroup up to 2048 tokens, and up to 4096 in 16-byte loads: no messages,
// and not the launch that clears them, which small vocabularies do not earn
// back.  Several workgroups -> one, us: every draft accepted, 1500 tokens 11.2 ->
// 8.8, 4000 11.1 -> 9.9; three rejections 16.0 -> 11.7, 15.1 -> 14.1; with rows of
// 4001 11.1 -> 11.4 and 17.3 -> 18.4, with 32 tokens a thread (8000) 11.4 -> 12.0
// and 16.7 -> 19.1, with 1024 threads instead slower still.  Above, 1024 tokens a
// workgroup while 64 of them reach, then twice as many; past 256 workgroups of
// 8192 one workgroup with p~ in memory.
template <bool SELECT>
hipError_t launch(const WalkIn &a, const TreeArg &tree, sb_step_result *result, int32_t *out,
                  void *ws, hipStream_t s, const WalkWait &wait) {
  double *arr = (double *)ws;  // 2 vocab float64: p~ in memory, then the messages
  unsigned long long *msg = (unsigned long long *)(arr + a.vocab);
  const int vec4 = (a.vocab & 3) == 0;
  auto go = [&](auto kernel, int grid, int threads) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, s, a, tree, vec4, wait, result, out, msg, arr);
    return hipGetLastError();
  };
  if (a.vocab <= 4 * kT) return go(k_walk<4, SELECT>, 1, kT);
  if (a.vocab <= 8 * kT) return go(k_walk<8, SELECT>, 1, kT);
  if (a.vocab <= 16 * kT && vec4) return go(k_walk<16, SELECT>, 1, kT);
  int ept = 4;
  while (ept < 32 && (a.vocab + kT * ept - 1) / (kT * ept) > 64) ept *= 2;
  const int G = (a.vocab - 1) / (kT * ept) + 1;
  if (G > kMaxG) return go(k_walk<0, SELECT>, 1, kMemT);
  hipLaunchKernelGGL(k_walk_clear, dim3(1), dim3(kT), 0, s, msg, 1 + 2 * G);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch (ept) {
    case 4: return go(k_walk<4, SELECT>, G, kT);
    case 8: return go(k_walk<8, SELECT>, G, kT);
    case 16: return go(k_walk<16, SELECT>, G, kT);
    default: return go(k_walk<32, SELECT>, G, kT);
  }
}

WalkIn walk_in(int vocab, int n, float temperature, const int32_t *tokens, const float *logits,
               const sb_row_stats *stats, const float *q, const float *u) {
  WalkIn a{};
  a.vocab = vocab;
  a.n = n;
  a.greedy = temperature <= 0.0f ? 1 : 0;
  a.inv_t = a.greedy ? 1.0f : 1.0f / temperature;
  a.tokens = tokens;
  a.logits = logits;
  a.stats = stats;
  a.q = q;
  a.u = u;
  return a;
}

}  // namespace

size_t sample_ws_bytes(int vocab) { return (size_t)2 * (size_t)vocab * sizeof(double); }

hipError_t launch_walk(int vocab, const TreeArg &tree, const int32_t *tokens, const float *logits,
                       const sb_row_stats *stats, float temperature, const float *q,
                       const float *u, sb_step_result *result, void *ws, hipStream_t s,
                       const WalkWait &wait) {
  return launch<false>(walk_in(vocab, tree.n, temperature, tokens, logits, stats, q, u), tree,
                       result, nullptr, ws, s, wait);
}

hipError_t launch_select(int vocab, const float *logits_row, const sb_row_stats *stats_row,
                         float temperature, int n_cand, const int32_t *cand_tokens,
                         const float *q, const float *u, int32_t *out, void *ws, hipStream_t s,
                         const WalkWait &wait) {
  WalkIn a = walk_in(vocab, n_cand + 1, temperature, cand_tokens, logits_row, stats_row, q, u);
  a.off = 1;
  a.u_draw = n_cand;
  const TreeArg none{};
  return launch<true>(a, none, nullptr, out, ws, s, wait);
}

}  // namespace sb
