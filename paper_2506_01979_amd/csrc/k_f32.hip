// float32 forward kernels, for the small exactness and parity shapes.
//
// At these sizes (hidden 64 .. 256, a few rows) a launch costs more than its
// work, so a layer is five of them: each projection carries what follows or
// precedes it (the RMSNorm of its input, RoPE and the cache writes, SwiGLU, the
// residual add), and a matrix is read once per 16 rows, not once per row.  The
// 2-layer shape of hidden 256 at 9 rows: 22 launches and 92 us as one kernel
// per operation, now 13 and 65 us.
#include <math.h>

#include "sb_device.h"
#include "sb_internal_fwd.h"

namespace sb {
namespace {

constexpr int kTokens = 16;  // rows of a projection workgroup
constexpr int kOuts = 16;    // outputs of it
constexpr int kWaves = 8;    // waves sharing its K
constexpr int kUnroll = 4;   // steps of a wave in flight

__device__ __forceinline__ float wave_sumf(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// E consecutive floats at p.
template <int E>
__device__ __forceinline__ void loadf(const float *p, float (&v)[E]) {
  if constexpr (E == 4) {
    const f32x4 t = *(const f32x4 *)p;
    v[0] = t[0], v[1] = t[1], v[2] = t[2], v[3] = t[3];
  } else {
    v[0] = *p;
  }
}

// Matrix row of output i (< kOuts) of workgroup u (invalid ones: any row).
// QKV: the RoPE pairs (j, j + d/2), j = 8 v .. 8 v + 7, of a q or k head
// (outputs i and i + 8), or 16 rows of v; SWIGLU: gate rows 8 u .. and the
// matching up rows.
template <int MODE>
__device__ __forceinline__ int out_row(const F32Args &a, int u, int i) {
  if constexpr (MODE == F32_QKV) {
    const int d = a.head_dim, per = d / 16, qk = (a.n_heads + a.n_kv) * per;
    if (u >= qk) return u * 16 + i;
    const int head = u / per, j = 8 * (u - head * per) + (i & 7);
    return head * d + j + (i >> 3) * (d / 2);
  } else if constexpr (MODE == F32_SWIGLU) {
    return (i >> 3) * a.M + min(8 * u + (i & 7), a.M - 1);
  } else {
    return min(u * kOuts + i, a.M - 1);
  }
}

// Y = X W^T for kTokens rows and kOuts outputs on the float32 matrix
// instruction: per step a lane loads E consecutive columns of one matrix row
// and of one X row straight into the operand registers, and E instructions
// multiply them.  The waves take the steps in turn and meet in LDS.  Bound by
// latency (one memory round trip, the LDS meeting, the launch), so the code is
// short: the same product as unrolled vector arithmetic took 8 us a launch,
// most of it instruction fetch, against 4.5 here.  QKV, SWIGLU and PLAIN
// read the residual h and apply its RMSNorm in factored form, r (h g) W^T.
template <int MODE, int E>
__global__ __launch_bounds__(kWaves * 64) void k_f32_proj(F32Args a) {
  constexpr bool NORM = MODE != F32_RESID;
  __shared__ float red[kWaves][kOuts][kTokens + 1], ssq[kWaves][kTokens];
  const int t0 = blockIdx.y * kTokens, nt = min(kTokens, a.n_tok - t0);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, l16 = lane & 15;
  const int kq = (lane >> 4) * E;  // this lane's first column within a step
  const float *wp = a.W + (size_t)out_row<MODE>(a, blockIdx.x, l16) * a.K;
  const float *xp = a.X + (size_t)(t0 + min(l16, nt - 1)) * a.K;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float ss = 0.0f;
  for (int k0 = w * 4 * E; k0 < a.K; k0 += kUnroll * kWaves * 4 * E) {
    float wv[kUnroll][E], xv[kUnroll][E], gv[kUnroll][E];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {  // columns past the end read the last ones, then count as zero
      const int k = min(k0 + u * kWaves * 4 * E + kq, a.K - E);
      loadf<E>(wp + k, wv[u]);
      loadf<E>(xp + k, xv[u]);
      if (NORM) loadf<E>(a.gain + k, gv[u]);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const bool in = k0 + u * kWaves * 4 * E + kq < a.K;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const float x = in ? xv[u][e] : 0.0f;
        if (NORM) ss += x * x;
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? wv[u][e] : 0.0f, NORM ? x * gv[u][e] : x,
                                                   acc, 0, 0, 0);
      }
    }
  }
  // lane: rows 4 (lane / 16) .. + 3 of token l16
#pragma unroll
  for (int i = 0; i < 4; ++i) red[w][4 * (lane >> 4) + i][l16] = acc[i];
  if (NORM) {
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    if (lane < 16) ssq[w][lane] = ss;
  }
  __syncthreads();
  auto sum = [&](int i, int t) {
    float v = red[0][i][t];
#pragma unroll
    for (int k = 1; k < kWaves; ++k) v += red[k][i][t];
    return v;
  };
  auto scale = [&](int t) {
    float v = ssq[0][t];
#pragma unroll
    for (int k = 1; k < kWaves; ++k) v += ssq[k][t];
    return 1.0f / sqrtf(v / (float)a.K + a.eps);
  };
  if constexpr (MODE == F32_RESID || MODE == F32_PLAIN) {
    const int i = threadIdx.x & 15, t = threadIdx.x >> 4, m = blockIdx.x * kOuts + i;
    if (t < nt && m < a.M) {
      float *y = a.Y + (size_t)(t0 + t) * a.M + m;
      *y = MODE == F32_RESID ? *y + sum(i, t) : sum(i, t) * scale(t);
    }
  } else {
    const int i = threadIdx.x & 7, t = threadIdx.x >> 3;
    if (t >= nt) return;
    const float r = scale(t), v1 = sum(i, t) * r, v2 = sum(i + 8, t) * r;
    const int tok = t0 + t;
    if constexpr (MODE == F32_SWIGLU) {
      const int f = 8 * blockIdx.x + i;
      if (f < a.M) a.Y[(size_t)tok * a.M + f] = v1 / (1.0f + expf(-v1)) * v2;
    } else {
      const int d = a.head_dim, per = d / 16, u = blockIdx.x;
      if (u < (a.n_heads + a.n_kv) * per) {
        const int head = u / per, j = 8 * (u - head * per) + i;
        const float2 cs = a.rope[tok * (d / 2) + j];
        float *dst = head < a.n_heads
                         ? a.Y + ((size_t)tok * a.n_heads + head) * d
                         : a.kc + ((size_t)(head - a.n_heads) * a.cap + a.kv_len + tok) * d;
        dst[j] = v1 * cs.x - v2 * cs.y;
        dst[j + d / 2] = v2 * cs.x + v1 * cs.y;
      } else {  // V is cached transposed: [head][d][slot], the heads' rows in turn
        const int m = (u - (a.n_heads + a.n_kv) * per) * 16 + i;
        a.vc[(size_t)m * a.cap + a.kv_len + tok] = v1;
        a.vc[(size_t)(m + 8) * a.cap + a.kv_len + tok] = v2;
      }
    }
  }
}

// One workgroup per (row t, query head): scores of every visible key in LDS
// (16 lanes a key, 32 keys of a wave in flight), softmax, then 8 dimensions of
// a wave at a time over the keys, lanes along the transposed V's slots.  The
// loads are branch-free (keys past the end read the last one and count as
// masked), so that a step's are all in flight.
template <int E>
__global__ __launch_bounds__(256) void k_f32_attn(AttnArgs a, float *__restrict__ out) {
  constexpr int UK = 8, UV = 2;
  extern __shared__ float sc[];  // [kv_len + n_tok]
  __shared__ __attribute__((aligned(16))) float sq[256];
  __shared__ float red[8];
  __shared__ uint32_t sanc[8];
  const int t = blockIdx.x, head = blockIdx.y;
  const int d = a.head_dim;
  const int G = a.n_heads / a.n_kv;
  const int g = head / G;
  const int nkeys = a.kv_len + a.n_tok;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const float *kc = (const float *)a.kc + (size_t)g * a.cap * d;
  const float *vt = (const float *)a.vc + (size_t)g * d * a.cap;  // [d][slot]
  if ((int)threadIdx.x < d)
    sq[threadIdx.x] = ((const float *)a.q)[((size_t)t * a.n_heads + head) * d + threadIdx.x];
  if (threadIdx.x < 8) sanc[threadIdx.x] = a.meta->anc[t][threadIdx.x];
  __syncthreads();
  float m = -INFINITY;
  const int l16 = lane & 15;
  for (int j0 = w * 4 + (lane >> 4); j0 < nkeys; j0 += 16 * UK) {
    float acc[UK];
#pragma unroll
    for (int u = 0; u < UK; ++u) acc[u] = 0.0f;
    for (int k = l16 * E; k < d; k += 16 * E) {
      float q[E], kv[UK][E];
#pragma unroll
      for (int u = 0; u < UK; ++u) loadf<E>(kc + (size_t)min(j0 + 16 * u, nkeys - 1) * d + k, kv[u]);
      loadf<E>(sq + k, q);
#pragma unroll
      for (int u = 0; u < UK; ++u)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[u] += q[e] * kv[u][e];
    }
#pragma unroll
    for (int b = 1; b < 16; b <<= 1)
#pragma unroll
      for (int u = 0; u < UK; ++u) acc[u] += __shfl_xor(acc[u], b, 64);
#pragma unroll
    for (int u = 0; u < UK; ++u) {
      const int j = j0 + 16 * u, jj = max(j - a.kv_len, 0) & (SB_MAX_ROWS - 1);
      const bool ok = j < nkeys && (j < a.kv_len || ((sanc[jj >> 5] >> (jj & 31)) & 1u));
      const float s = ok ? acc[u] * a.scale : -INFINITY;
      if (l16 == 0 && j < nkeys) sc[j] = s;
      m = fmaxf(m, s);
    }
  }
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  if (lane == 0) red[w] = m;
  __syncthreads();
  m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  float l = 0.0f;
  for (int j = threadIdx.x; j < nkeys; j += 256) {
    const float e = expf(sc[j] - m);
    sc[j] = e;
    l += e;
  }
  l = wave_sumf(l);
  if (lane == 0) red[4 + w] = l;
  __syncthreads();
  l = red[4] + red[5] + red[6] + red[7];
  for (int d0 = w * 8; d0 < d; d0 += 32) {
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.0f;
    const float *vr = vt + (size_t)d0 * a.cap;
    for (int j0 = lane; j0 < nkeys; j0 += 64 * UV) {
      float v[UV][8];
#pragma unroll
      for (int u = 0; u < UV; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i) v[u][i] = vr[(size_t)i * a.cap + min(j0 + 64 * u, nkeys - 1)];
#pragma unroll
      for (int u = 0; u < UV; ++u) {
        const float p = j0 + 64 * u < nkeys ? sc[min(j0 + 64 * u, nkeys - 1)] : 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += p * v[u][i];
      }
    }
#pragma unroll
    for (int b = 32; b > 0; b >>= 1)
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += __shfl_xor(acc[i], b, 64);
    float o = acc[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) o = lane == i ? acc[i] : o;
    if (lane < 8) out[(size_t)t * a.n_heads * d + (size_t)head * d + d0 + lane] = o / l;
  }
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

hipError_t launch_f32_proj(int mode, const F32Args &a, hipStream_t s) {
  int units = (a.M + kOuts - 1) / kOuts;
  if (mode == F32_QKV) units = (a.n_heads + 2 * a.n_kv) * (a.head_dim / 16);
  if (mode == F32_SWIGLU) units = (a.M + 7) / 8;
  const dim3 grid(units, (a.n_tok + kTokens - 1) / kTokens), block(kWaves * 64);
  // 16-byte loads where every row starts on 16 bytes
  const bool vec = a.K % 4 == 0 && aligned16(a.W) && aligned16(a.X) && aligned16(a.gain);
  switch (mode) {
#define SB_MODE(m)                                                                 \
  case m:                                                                          \
    if (vec)                                                                       \
      hipLaunchKernelGGL((k_f32_proj<m, 4>), grid, block, 0, s, a);                \
    else                                                                           \
      hipLaunchKernelGGL((k_f32_proj<m, 1>), grid, block, 0, s, a);                \
    break;
    SB_MODE(F32_QKV) SB_MODE(F32_RESID) SB_MODE(F32_SWIGLU) SB_MODE(F32_PLAIN)
#undef SB_MODE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_f32_attn(const AttnArgs &a, float *out, hipStream_t s) {
  if (a.head_dim > 256 || a.head_dim % 16 != 0) return hipErrorInvalidValue;
  const size_t lds = (size_t)(a.kv_len + a.n_tok) * sizeof(float);
  dim3 grid(a.n_tok, a.n_heads);
  if (aligned16(a.kc))
    hipLaunchKernelGGL(k_f32_attn<4>, grid, dim3(256), lds, s, a, out);
  else
    hipLaunchKernelGGL(k_f32_attn<1>, grid, dim3(256), lds, s, a, out);
  return hipGetLastError();
}

}  // namespace sb
