// Row softmax statistics and the draft's rows and draws.
//
// What is computed:
//   p(v) = fl32(exp(fl32(fl32(l_v * fl32(1/T)) - zmax))) / total  (float64)
//          or the one-hot at argmax when T = 0;
//   draw : C_v = running float64 sum in vocabulary order,
//          y = min{v : C_v > u * W}, W the float64 total; a zero-mass
//          token is never drawn.
// The multiply-then-subtract of the logit transform must not be contracted
// into an FMA: every operation rounds on its own, as the definition states.
#pragma clang fp contract(off)

#include <float.h>
#include <limits.h>
#include <math.h>

#include "sb_device.h"
#include "sb_internal.h"

namespace sb {
namespace {

constexpr int kRowThreads = 1024;
constexpr int kRowWaves = kRowThreads / 64;

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Block-wide reductions for blockDim.x == nthreads (multiple of 64).
template <int NW>
__device__ double block_sum(double v, double *red) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  v = wave_sum(v);
  if (lane == 0) red[w] = v;
  __syncthreads();
  double t = 0.0;
  if (w == 0) {
    t = lane < NW ? red[lane] : 0.0;
    t = wave_sum(t);
    if (lane == 0) red[NW] = t;
  }
  __syncthreads();
  t = red[NW];
  __syncthreads();
  return t;
}

// One workgroup per row.  Pass 1: max of l (lowest-index argmax), max of
// z = fl32(l / T) and a NaN/+inf scan; pass 2: float64 sum of
// fl32(exp(z - zmax)).  Loads are 16-byte and independent across a thread's
// items so a pass costs about one memory latency.
// Row statistics with the whole row in registers (vocab a multiple of 4 and
// at most NB * 4096): one read of the row, the max / argmax / non-finite
// scan and the exp sum both run on the registers.
template <int NB>
__global__ __launch_bounds__(1024) void k_softmax_stats_reg(const float *__restrict__ logits,
                                                            int vocab, float inv_t, int greedy,
                                                            sb_row_stats *__restrict__ out,
                                                            const unsigned *invalid) {
  constexpr int NT = 1024, NW = NT / 64;
  __shared__ float smax[NW], szmax[NW];
  __shared__ int sarg[NW];
  __shared__ int sbad[NW];
  __shared__ double red[NW];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int n4 = vocab >> 2;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(logits + (size_t)blockIdx.x * vocab), 0, vocab * 4, kBufferDword3);
  f32x4 x[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int i = threadIdx.x + j * NT;
    x[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, i * 16, 0, 0));
  }
  float best = -INFINITY;
  int barg = INT_MAX;
  float zbest = -INFINITY;
  int bad = 0;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int i = threadIdx.x + j * NT;
    if (i < n4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = x[j][e];
        if (isnan(v) || v == INFINITY) bad = 1;
        if (v > best) {
          best = v;
          barg = 4 * i + e;
        }
        zbest = fmaxf(zbest, v * inv_t);
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const float ob = __shfl_xor(best, o, 64);
    const int oa = __shfl_xor(barg, o, 64);
    if (ob > best || (ob == best && oa < barg)) {
      best = ob;
      barg = oa;
    }
    zbest = fmaxf(zbest, __shfl_xor(zbest, o, 64));
    bad |= __shfl_xor(bad, o, 64);
  }
  if (lane == 0) {
    smax[w] = best;
    sarg[w] = barg;
    sbad[w] = bad;
    szmax[w] = zbest;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float b = smax[0], zb = szmax[0];
    int a = sarg[0], bd = sbad[0];
    for (int i = 1; i < NW; ++i) {
      if (smax[i] > b || (smax[i] == b && sarg[i] < a)) {
        b = smax[i];
        a = sarg[i];
      }
      zb = fmaxf(zb, szmax[i]);
      bd |= sbad[i];
    }
    smax[0] = greedy ? b : zb;
    sarg[0] = (a == INT_MAX) ? 0 : a;
    sbad[0] = bd;
  }
  __syncthreads();
  const float zmax = smax[0];
  const int arg = sarg[0];
  const int anybad = sbad[0];
  double total = 1.0;
  if (!greedy) {
    double part = 0.0;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int i = threadIdx.x + j * NT;
      if (i < n4)
#pragma unroll
        for (int e = 0; e < 4; ++e) part += (double)expf(x[j][e] * inv_t - zmax);
    }
    part = wave_sum(part);
    if (lane == 0) red[w] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int i = 0; i < NW; ++i) t += red[i];
      red[0] = t;
    }
    __syncthreads();
    total = red[0];
  }
  if (threadIdx.x == 0) {
    sb_row_stats st;
    st.zmax = zmax;
    st.argmax = arg;
    // a producer that flagged the logits invalid makes the row non-finite
    st.total = (anybad || (invalid && *invalid != 0u)) ? (double)NAN : total;
    out[blockIdx.x] = st;
  }
}

// The statistics of row blockIdx.x from its groups' partials (the LM
// head's workgroups, at most 256): the largest logit and its lowest index
// over the groups, zmax = fl32(lmax / T) (rounding is monotone, so this is
// the largest scaled logit), and total = the float64 sum over groups of
// sum_g exp(m_g - zmax), m_g = fl32(lmax_g / T), in a fixed order.  A row
// with nothing above -inf has a NaN total at T > 0, as exp(-inf - -inf).
__global__ __launch_bounds__(256) void k_softmax_stats_finish(const LmPart *__restrict__ part,
                                                             int groups, float inv_t, int greedy,
                                                             sb_row_stats *__restrict__ out) {
  constexpr int NW = 256 / 64;
  __shared__ float sbest[NW];
  __shared__ int sarg[NW];
  __shared__ double red[NW + 1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  LmPart p{-INFINITY, INT_MAX, 0.0};
  if ((int)threadIdx.x < groups) p = part[(size_t)blockIdx.x * groups + threadIdx.x];
  float best = p.lmax;
  int arg = p.arg;
  for (int o = 32; o > 0; o >>= 1) {
    const float ob = __shfl_xor(best, o, 64);
    const int oa = __shfl_xor(arg, o, 64);
    if (ob > best || (ob == best && oa < arg)) {
      best = ob;
      arg = oa;
    }
  }
  if (lane == 0) {
    sbest[w] = best;
    sarg[w] = arg;
  }
  __syncthreads();
  best = sbest[0];
  arg = sarg[0];
  for (int i = 1; i < NW; ++i)
    if (sbest[i] > best || (sbest[i] == best && sarg[i] < arg)) {
      best = sbest[i];
      arg = sarg[i];
    }
  const float zmax = greedy ? best : best * inv_t;
  double term = p.sum;
  if (!greedy && p.sum != 0.0) term = p.sum * exp((double)(p.lmax * inv_t) - (double)zmax);
  const double s = block_sum<NW>(term, red);
  if (threadIdx.x == 0) {
    sb_row_stats st;
    st.zmax = zmax;
    st.argmax = arg == INT_MAX ? 0 : arg;
    if (greedy)
      st.total = isnan(s) ? (double)NAN : 1.0;
    else
      st.total = best == -INFINITY ? (double)NAN : s;
    out[blockIdx.x] = st;
  }
}

__global__ __launch_bounds__(1024) void k_softmax_stats(const float *__restrict__ logits,
                                                        int vocab, float inv_t, int greedy,
                                                        sb_row_stats *__restrict__ out,
                                                            const unsigned *invalid) {
  constexpr int NT = 1024, NW = NT / 64;
  __shared__ float smax[NW], szmax[NW];
  __shared__ int sarg[NW];
  __shared__ int sbad[NW];
  __shared__ double red[NW];
  const float *l = logits + (size_t)blockIdx.x * vocab;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const bool vec = (vocab & 3) == 0;
  float best = -INFINITY;
  int barg = INT_MAX;
  float zbest = -INFINITY;
  int bad = 0;
  auto visit = [&](float x, int v) {
    if (isnan(x) || x == INFINITY) bad = 1;
    if (x > best) {
      best = x;
      barg = v;
    }
    zbest = fmaxf(zbest, x * inv_t);
  };
  if (vec) {
    const float4 *l4 = (const float4 *)l;
    const int n4 = vocab >> 2;
    for (int i0 = threadIdx.x; i0 < n4; i0 += 4 * NT) {
      float4 x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        x[j] = (i0 + j * NT < n4) ? l4[i0 + j * NT] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = i0 + j * NT;
        if (i < n4) {
          visit(x[j].x, 4 * i);
          visit(x[j].y, 4 * i + 1);
          visit(x[j].z, 4 * i + 2);
          visit(x[j].w, 4 * i + 3);
        }
      }
    }
  } else {
    for (int v = threadIdx.x; v < vocab; v += NT) visit(l[v], v);
  }
  for (int o = 32; o > 0; o >>= 1) {
    const float ob = __shfl_xor(best, o, 64);
    const int oa = __shfl_xor(barg, o, 64);
    if (ob > best || (ob == best && oa < barg)) {
      best = ob;
      barg = oa;
    }
    zbest = fmaxf(zbest, __shfl_xor(zbest, o, 64));
    bad |= __shfl_xor(bad, o, 64);
  }
  if (lane == 0) {
    smax[w] = best;
    sarg[w] = barg;
    sbad[w] = bad;
    szmax[w] = zbest;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float b = smax[0], zb = szmax[0];
    int a = sarg[0], bd = sbad[0];
    for (int i = 1; i < NW; ++i) {
      if (smax[i] > b || (smax[i] == b && sarg[i] < a)) {
        b = smax[i];
        a = sarg[i];
      }
      zb = fmaxf(zb, szmax[i]);
      bd |= sbad[i];
    }
    smax[0] = greedy ? b : zb;
    sarg[0] = (a == INT_MAX) ? 0 : a;
    sbad[0] = bd;
  }
  __syncthreads();
  const float zmax = smax[0];
  const int arg = sarg[0];
  const int anybad = sbad[0];
  double total = 1.0;
  if (!greedy) {
    double part = 0.0;
    if (vec) {
      const float4 *l4 = (const float4 *)l;
      const int n4 = vocab >> 2;
      for (int i0 = threadIdx.x; i0 < n4; i0 += 4 * NT) {
        float4 x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          x[j] = (i0 + j * NT < n4) ? l4[i0 + j * NT] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          part += (double)expf(x[j].x * inv_t - zmax);
          part += (double)expf(x[j].y * inv_t - zmax);
          part += (double)expf(x[j].z * inv_t - zmax);
          part += (double)expf(x[j].w * inv_t - zmax);
        }
      }
    } else {
      for (int v = threadIdx.x; v < vocab; v += NT) part += (double)expf(l[v] * inv_t - zmax);
    }
    part = wave_sum(part);
    if (lane == 0) red[w] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int i = 0; i < NW; ++i) t += red[i];
      red[0] = t;
    }
    __syncthreads();
    total = red[0];
  }
  if (threadIdx.x == 0) {
    sb_row_stats st;
    st.zmax = zmax;
    st.argmax = arg;
    // a producer that flagged the logits invalid makes the row non-finite
    st.total = (anybad || (invalid && *invalid != 0u)) ? (double)NAN : total;
    out[blockIdx.x] = st;
  }
}

// The draft's rows (the draft side of a round): q(v) = float32(p(v)) of a
// logits row at T, written out as the row verification later reads as q,
// and the token drawn from those float32 values: their float64 running sum
// in vocabulary order, the first v whose sum exceeds u * W.  T = 0: q is
// one-hot at the row's argmax, which is the token.
//   k_draft_q:    grid (blocks of kDraftSpan tokens, rows); writes q and the
//                 float64 sum of each block's q to the workspace;
//   k_draft_draw: one workgroup per row; the crossing block from the block
//                 sums, then the token from that block's q.
constexpr int kDraftThreads = 256;
constexpr int kDraftSpan = kDraftThreads * 8;

__device__ __forceinline__ float draft_qv(float raw, float inv_t, float zmax, double total) {
  const float z = raw * inv_t;
  const float e = expf(z - zmax);
  return (float)((double)e / total);
}

__global__ __launch_bounds__(kDraftThreads) void k_draft_q(int vocab, int vec8, DraftRows rows,
                                                           const float *__restrict__ logits,
                                                           const sb_row_stats *__restrict__ stats,
                                                           float inv_t, int greedy,
                                                           float *__restrict__ q,
                                                           double *__restrict__ bsum) {
  __shared__ double red[kDraftThreads / 64];
  const int i = blockIdx.y, blk = blockIdx.x, nblk = gridDim.x;
  const int src = rows.src[i], dst = rows.dst[i];
  const float *l = logits + (size_t)src * vocab;
  const sb_row_stats st = stats[src];
  float *qr = q + (size_t)dst * vocab;
  // thread t: the 8 consecutive tokens v0 .. v0 + 7 of the block (whole
  // 16-byte pairs when vocab % 8 == 0 and the rows are 16-byte aligned)
  const int v0 = blk * kDraftSpan + (int)threadIdx.x * 8;
  float raw[8];
  if (vec8 && v0 < vocab) {
    const f32x4 a = *(const f32x4 *)(l + v0), b = *(const f32x4 *)(l + v0 + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      raw[e] = a[e];
      raw[4 + e] = b[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) raw[e] = v0 + e < vocab ? l[v0 + e] : 0.0f;
  }
  float f[8];
  double part = 0.0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int v = v0 + e;
    f[e] = greedy ? (v == st.argmax ? 1.0f : 0.0f) : draft_qv(raw[e], inv_t, st.zmax, st.total);
    if (v < vocab) part += (double)f[e];
  }
  if (vec8 && v0 < vocab) {
    *(f32x4 *)(qr + v0) = f32x4{f[0], f[1], f[2], f[3]};
    *(f32x4 *)(qr + v0 + 4) = f32x4{f[4], f[5], f[6], f[7]};
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (v0 + e < vocab) qr[v0 + e] = f[e];
  }
  part = wave_sum(part);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = part;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = red[0];
    for (int w = 1; w < kDraftThreads / 64; ++w) t += red[w];
    bsum[(size_t)i * nblk + blk] = t;
  }
}

// Inclusive 64-lane scan of a double.
__device__ __forceinline__ double wave_scan(double x) {
  const int lane = threadIdx.x & 63;
  for (int o = 1; o < 64; o <<= 1) {
    const double y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

__global__ __launch_bounds__(kDraftThreads) void k_draft_draw(int vocab, int nblk, DraftRows rows,
                                                              const sb_row_stats *__restrict__ stats,
                                                              int greedy, const float *__restrict__ u,
                                                              int32_t *__restrict__ tokens,
                                                              const float *__restrict__ q,
                                                              const double *__restrict__ bsum,
                                                              float *__restrict__ conf) {
  __shared__ double s_base, s_thr, wsum[kDraftThreads / 64];
  __shared__ int s_blk, s_tok;
  const int i = blockIdx.x;
  const int src = rows.src[i], dst = rows.dst[i];
  if (greedy) {
    if (threadIdx.x == 0) {
      tokens[dst] = stats[src].argmax;
      if (conf) conf[i] = 1.0f;
    }
    return;
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double *bs = bsum + (size_t)i * nblk;
  // wave 0: lane l sums the block sums l*per .. l*per + per - 1 in order,
  // scans the lane sums, and finds the first block whose running sum
  // exceeds u * W (else the last block with mass)
  if (w == 0) {
    const int per = (nblk + 63) / 64;
    double ls = 0.0;
    for (int j = 0; j < per; ++j) {
      const int b = lane * per + j;
      if (b < nblk) ls += bs[b];
    }
    const double inc = wave_scan(ls);
    const double W = __shfl(inc, 63, 64);
    const double thr = (double)u[i] * W;
    const unsigned long long hit = __ballot(ls > 0.0 && inc > thr);
    int sel_lane;
    if (hit) {
      sel_lane = __ffsll((long long)hit) - 1;
    } else {
      const unsigned long long pos = __ballot(ls > 0.0);
      sel_lane = pos ? 63 - __clzll((long long)pos) : 0;
    }
    if (lane == sel_lane) {
      double run = inc - ls;
      int blk = -1, last = -1;
      double base_at = run, base_last = run;
      for (int j = 0; j < per; ++j) {
        const int b = lane * per + j;
        if (b >= nblk) break;
        const double x = bs[b];
        if (x > 0.0) {
          last = b;
          base_last = run;
          if (blk < 0 && run + x > thr) {
            blk = b;
            base_at = run;
          }
        }
        run += x;
      }
      if (blk < 0) {
        blk = last < 0 ? 0 : last;
        base_at = base_last;
      }
      s_blk = blk;
      s_base = base_at;
      s_thr = thr;
    }
  }
  __syncthreads();
  // the crossing block: thread t holds its 8 consecutive values, a block-wide
  // scan of the thread sums finds the thread, that thread finds the token
  const int blk = s_blk;
  const double thr = s_thr - s_base;
  const int v0 = blk * kDraftSpan + (int)threadIdx.x * 8;
  const float *qr = q + (size_t)dst * vocab;
  double x[8], ts = 0.0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    x[e] = v0 + e < vocab ? (double)qr[v0 + e] : 0.0;
    ts += x[e];
  }
  const double inc = wave_scan(ts);
  if (lane == 63) wsum[w] = inc;
  if (threadIdx.x == 0) s_tok = INT_MAX;
  __syncthreads();
  double off = 0.0;
  for (int k = 0; k < w; ++k) off += wsum[k];
  const double start = off + inc - ts;
  const unsigned long long hit = __ballot(ts > 0.0 && start + ts > thr);
  int found = INT_MAX;
  if (hit && lane == __ffsll((long long)hit) - 1) {
    double c = start;
    for (int e = 0; e < 8; ++e) {
      c += x[e];
      if (x[e] > 0.0 && c > thr) {
        found = v0 + e;
        break;
      }
    }
    if (found == INT_MAX)  // rounding: the thread's last token with mass
      for (int e = 0; e < 8; ++e)
        if (x[e] > 0.0) found = v0 + e;
  }
  if (found != INT_MAX) atomicMin(&s_tok, found);
  __syncthreads();
  if (threadIdx.x == 0) {
    int y = s_tok;
    if (y == INT_MAX) {
      // rounding left no crossing in the block: its last token with mass
      for (int v = min(vocab, (blk + 1) * kDraftSpan) - 1; v >= blk * kDraftSpan; --v)
        if (qr[v] > 0.0f) {
          y = v;
          break;
        }
      if (y == INT_MAX) y = stats[src].argmax;
    }
    tokens[dst] = y;
    if (conf) conf[i] = qr[y];  // the drawn token's own probability
  }
}

// A chain draft's q row conditioned on confidence, in place: q(v) / q(C)
// on C = {v : q(v) >= eps} (float32 comparisons), zero elsewhere, with q(C)
// the float64 sum of C's float32 values and each quotient rounded once to
// float32.  A row with no confident token is left all zero.
__global__ __launch_bounds__(kRowThreads) void k_confident_row(float *q, int vocab, float eps) {
  __shared__ double red[kRowWaves + 1];
  double part = 0.0;
  for (int v = threadIdx.x; v < vocab; v += kRowThreads) {
    const float x = q[v];
    if (x >= eps) part += (double)x;
  }
  const double mass = block_sum<kRowWaves>(part, red);
  for (int v = threadIdx.x; v < vocab; v += kRowThreads) {
    const float x = q[v];
    q[v] = x >= eps && mass > 0.0 ? (float)((double)x / mass) : 0.0f;
  }
}

}  // namespace

hipError_t launch_confident_row(float *q, int vocab, float eps, hipStream_t s) {
  hipLaunchKernelGGL(k_confident_row, dim3(1), dim3(kRowThreads), 0, s, q, vocab, eps);
  return hipGetLastError();
}

static inline void temp_args(float temperature, float *inv_t, int *greedy) {
  *greedy = temperature <= 0.0f ? 1 : 0;
  *inv_t = *greedy ? 1.0f : 1.0f / temperature;
}

hipError_t launch_softmax_stats(int vocab, int n_rows, const float *logits, float temperature,
                                sb_row_stats *stats, hipStream_t s, const unsigned *invalid) {
  float inv_t;
  int greedy;
  temp_args(temperature, &inv_t, &greedy);
  const int nb = (vocab + 4095) / 4096;  // float4 per thread with the row in registers
  if ((vocab & 3) == 0 && nb <= 16) {
#define SB_NB(k)                                                                                  \
  if (nb <= k) {                                                                                  \
    hipLaunchKernelGGL(k_softmax_stats_reg<k>, dim3(n_rows), dim3(1024), 0, s, logits, vocab,     \
                       inv_t, greedy, stats, invalid);                                            \
    return hipGetLastError();                                                                     \
  }
    SB_NB(1) SB_NB(2) SB_NB(4) SB_NB(8) SB_NB(16)
#undef SB_NB
  }
  hipLaunchKernelGGL(k_softmax_stats, dim3(n_rows), dim3(1024), 0, s, logits, vocab, inv_t, greedy,
                     stats, invalid);
  return hipGetLastError();
}

hipError_t launch_stats_finish(const LmPart *part, int groups, int n_rows, float temperature,
                               sb_row_stats *stats, hipStream_t s) {
  if (groups < 1 || groups > 256 || n_rows < 1) return hipErrorInvalidValue;
  float inv_t;
  int greedy;
  temp_args(temperature, &inv_t, &greedy);
  hipLaunchKernelGGL(k_softmax_stats_finish, dim3(n_rows), dim3(256), 0, s, part, groups, inv_t,
                     greedy, stats);
  return hipGetLastError();
}

size_t draft_ws_bytes(int vocab, int n) {
  return (size_t)n * ((vocab + kDraftSpan - 1) / kDraftSpan) * sizeof(double);
}

hipError_t launch_draft_sample(int vocab, const DraftRows &rows, const float *logits,
                               const sb_row_stats *stats, float temperature, const float *u,
                               int32_t *tokens, float *q, void *ws, hipStream_t s, float *conf) {
  float inv_t;
  int greedy;
  temp_args(temperature, &inv_t, &greedy);
  const int nblk = (vocab + kDraftSpan - 1) / kDraftSpan;
  const int vec8 = vocab % 8 == 0 && ((uintptr_t)logits & 15) == 0 && ((uintptr_t)q & 15) == 0;
  hipLaunchKernelGGL(k_draft_q, dim3(nblk, rows.n), dim3(kDraftThreads), 0, s, vocab, vec8, rows,
                     logits, stats, inv_t, greedy, q, (double *)ws);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_draft_draw, dim3(rows.n), dim3(kDraftThreads), 0, s, vocab, nblk, rows,
                     stats, greedy, u, tokens, q, (const double *)ws, conf);
  return hipGetLastError();
}

}  // namespace sb
