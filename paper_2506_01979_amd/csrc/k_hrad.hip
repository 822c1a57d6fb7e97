// H-RAD's draft-length predictor (Section "H-RAD", equations for z_t and
// s_t): the features are the target's residual stream after each of its
// last K layers at the last accepted row, concatenated with the embedding
// of the new token; a 256/64/3 ReLU MLP maps them to three logits, and the
// class is their argmax (softmax is monotone).  float32 arithmetic.
#include "sb_device.h"
#include "sb_internal_fwd.h"

namespace sb {
namespace {

constexpr int kL1Threads = 256;
constexpr int kL1Batch = 20;  // 16-byte loads of W1 in flight per thread
constexpr int kTailThreads = 512;

// The row and token the features come from: the last row of the walk's
// path and its next token; false when the result names no usable pair.
__device__ __forceinline__ bool hrad_source(const HradArgs &a, int *row, int *tok) {
  const int plen = a.res->path_len;
  if (plen < 1 || plen > SB_MAX_ROWS) return false;
  const int r = a.res->path[plen - 1];
  const int y = a.res->next_token;
  if (r < 0 || r >= a.max_rows || y < 0 || y >= a.vocab) return false;
  *row = r;
  *tok = y;
  return true;
}

// One workgroup per unit j of the first layer: y1[j] = ReLU(W1[j] . z + b1[j]),
// z = (tap 0 .. tap k-1 of the row, the token's embedding); a thread takes 4
// consecutive inputs per step (hidden is a multiple of 8, so 4 never straddle
// two parts of z).  Bound by W1 from memory (21 MB at hidden 4096 and 4 taps):
// the weights of kL1Batch steps go out before the row and the token, a chain
// of three dependent reads, are looked up.  A batch is 20480 inputs; wider
// features take the rest after it, narrower ones read past the row's end (zero,
// no traffic).  Both launches, host to host, against loads as they are needed:
// 4 taps at hidden 512 to 4096 14.5 -> 12 us, at 5120 (25 steps) 18 -> 12, at
// 8192 (40) 27 -> 17.
__global__ __launch_bounds__(kL1Threads) void k_hrad_l1(HradArgs a) {
  __shared__ float red[kL1Threads / 64];
  const int j = blockIdx.x;
  const int H = a.hidden;
  const int din = (a.k + 1) * H;
  const __amdgpu_buffer_rsrc_t wrs = uniform_rsrc(a.w1 + (size_t)j * din, din * 4);
  f32x4 wv[kL1Batch];
  auto load_w = [&](int i0) {
#pragma unroll
    for (int b = 0; b < kL1Batch; ++b)
      wv[b] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                            wrs, (i0 + b * kL1Threads * 4) * 4, 0, 0));
  };
  const int first = (int)threadIdx.x * 4;
  load_w(first);
  __builtin_amdgcn_sched_barrier(0);
  int r = 0, y = 0;
  const bool ok = hrad_source(a, &r, &y);
  float acc = 0.0f;
  if (ok) {
    for (int i0 = first; i0 < din; i0 += kL1Batch * kL1Threads * 4) {
      if (i0 != first) load_w(i0);
#pragma unroll
      for (int b = 0; b < kL1Batch; ++b) {
        const int i = i0 + b * kL1Threads * 4;
        f32x4 zv = {0.f, 0.f, 0.f, 0.f};
        if (i < din) {
          const int k = i / H, d = i - k * H;
          if (k < a.k) {
            zv = *(const f32x4 *)(a.taps + ((size_t)k * a.max_rows + r) * H + d);
          } else {
            const uint2 e = *(const uint2 *)(a.embed + (size_t)y * H + d);
            zv = f32x4{bf2f((uint16_t)(e.x & 0xffff)), bf2f((uint16_t)(e.x >> 16)),
                       bf2f((uint16_t)(e.y & 0xffff)), bf2f((uint16_t)(e.y >> 16))};
          }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) acc += wv[b][c] * zv[c];
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float sum = red[0];
#pragma unroll
    for (int w = 1; w < kL1Threads / 64; ++w) sum += red[w];
    a.y1[j] = ok ? fmaxf(sum + a.b1[j], 0.0f) : 0.0f;
  }
}

// The 64-unit layer (thread m computes unit m), then the 3 logits (one thread
// each) and their argmax (lowest index on ties).  Bound by latency: W2 and W3
// go to LDS by all threads at once, and only the sums, whose order is fixed,
// are serial.
__global__ __launch_bounds__(kTailThreads) void k_hrad_tail(HradArgs a) {
  constexpr int LD = SB_HRAD_H1 + 4;  // row of W2 in LDS: rows start 4 banks apart
  constexpr int W2V = SB_HRAD_H2 * SB_HRAD_H1 / 4, PER = W2V / kTailThreads;
  static_assert(PER * kTailThreads == W2V && SB_HRAD_H1 <= kTailThreads, "whole pieces");
  static_assert(SB_HRAD_CLASSES * SB_HRAD_H2 <= kTailThreads, "one W3 value per thread");
  __shared__ __attribute__((aligned(16))) float w2[SB_HRAD_H2 * LD];
  __shared__ __attribute__((aligned(16))) float y1[SB_HRAD_H1];
  __shared__ float w3[SB_HRAD_CLASSES * SB_HRAD_H2], y2[SB_HRAD_H2], lg[SB_HRAD_CLASSES];
  const int tid = threadIdx.x;
  const __amdgpu_buffer_rsrc_t wrs = uniform_rsrc(a.w2, SB_HRAD_H2 * SB_HRAD_H1 * 4);
  f32x4 wv[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i)
    wv[i] = __builtin_bit_cast(
        f32x4, __builtin_amdgcn_raw_buffer_load_b128(wrs, (i * kTailThreads + tid) * 16, 0, 0));
  const float w3v = tid < SB_HRAD_CLASSES * SB_HRAD_H2 ? a.w3[tid] : 0.0f;
  const float y1v = tid < SB_HRAD_H1 ? a.y1[tid] : 0.0f;
  const float b2 = tid < SB_HRAD_H2 ? a.b2[tid] : 0.0f;
  const float b3 = tid < SB_HRAD_CLASSES ? a.b3[tid] : 0.0f;
  int r = 0, y = 0;
  const bool ok = hrad_source(a, &r, &y);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int at = (i * kTailThreads + tid) * 4;
    *(f32x4 *)&w2[at / SB_HRAD_H1 * LD + at % SB_HRAD_H1] = wv[i];
  }
  if (tid < SB_HRAD_CLASSES * SB_HRAD_H2) w3[tid] = w3v;
  if (tid < SB_HRAD_H1) y1[tid] = y1v;
  __syncthreads();
  if (tid < SB_HRAD_H2) {
    float acc = 0.0f;
#pragma unroll 16
    for (int i = 0; i < SB_HRAD_H1; i += 4) {
      const f32x4 w = *(const f32x4 *)&w2[tid * LD + i], v = *(const f32x4 *)&y1[i];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc += w[c] * v[c];
    }
    y2[tid] = fmaxf(acc + b2, 0.0f);
  }
  __syncthreads();
  if (tid < SB_HRAD_CLASSES) {
    float acc = 0.0f;
#pragma unroll 16
    for (int i = 0; i < SB_HRAD_H2; ++i) acc += w3[tid * SB_HRAD_H2 + i] * y2[i];
    lg[tid] = acc + b3;
  }
  __syncthreads();
  if (tid == 0) {
    int best = 0;
    for (int c = 1; c < SB_HRAD_CLASSES; ++c)
      if (lg[c] > lg[best]) best = c;
    for (int c = 0; c < SB_HRAD_CLASSES; ++c) a.logits3[c] = ok ? lg[c] : 0.0f;
    *a.cls = ok ? best : -1;
  }
}

}  // namespace

hipError_t launch_hrad(const HradArgs &a, hipStream_t s) {
  if (a.hidden % 8 != 0 || a.k < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_hrad_l1, dim3(SB_HRAD_H1), dim3(kL1Threads), 0, s, a);
  hipLaunchKernelGGL(k_hrad_tail, dim3(1), dim3(kTailThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace sb
