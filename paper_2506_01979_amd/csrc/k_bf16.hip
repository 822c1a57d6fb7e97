// bf16 forward kernels for gfx950 other than the GEMM: weight packing,
// embedding + tree metadata + RoPE table, and RMSNorm of the fp32 residual
// rows into the packed operand layout of the GEMM.
#include <math.h>

#include "sb_device.h"
#include "sb_internal_fwd.h"

namespace sb {
namespace {

static_assert(SB_MAX_ROWS == 256, "k_embed_meta: one thread per row, four waves");

// ---------------------------------------------------------------------------
// packing
// ---------------------------------------------------------------------------

struct PackArgs {
  const uint16_t *src0, *src1, *src2;
  uint16_t *dst;
  int kind;
  int K;        // source columns
  int ks;       // packed k-steps (K padded to whole 8-k-step chunks)
  int tiles;
  int n_heads, n_kv, head_dim, ffn, rows0;  // rows0: rows of src0 for O/DOWN/LM
};

// Source row of tile row r: returns the matrix and row, or nullptr.
__device__ const uint16_t *pack_src_row(const PackArgs &a, int tile, int r) {
  switch (a.kind) {
    case SB_W_QKV: {
      const int d = a.head_dim, ht = d / 16;
      const int qt = a.n_heads * ht, kt = a.n_kv * ht;
      if (tile < qt + kt) {
        const uint16_t *m = tile < qt ? a.src0 : a.src1;
        const int idx = tile < qt ? tile : tile - qt;
        const int head = idx / ht, u = idx % ht;
        const int dim = r < 8 ? 8 * u + r : d / 2 + 8 * u + (r - 8);
        return m + (size_t)(head * d + dim) * a.K;
      }
      const int idx = tile - qt - kt;
      const int row = idx * 16 + r;
      if (row >= a.n_kv * d) return nullptr;
      return a.src2 + (size_t)row * a.K;
    }
    case SB_W_GATE_UP: {
      const int f = tile * 8 + (r & 7);
      if (f >= a.ffn) return nullptr;
      return (r < 8 ? a.src0 : a.src1) + (size_t)f * a.K;
    }
    default: {
      const int row = tile * 16 + r;
      if (row >= a.rows0) return nullptr;
      return a.src0 + (size_t)row * a.K;
    }
  }
}

__global__ __launch_bounds__(256) void k_pack(PackArgs a) {
  const size_t total = (size_t)a.tiles * a.ks * 64;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (size_t)gridDim.x * blockDim.x) {
    const int lane = (int)(i & 63);
    const size_t ts = i >> 6;
    const int s = (int)(ts % a.ks);
    const int tile = (int)(ts / a.ks);
    const uint16_t *row = pack_src_row(a, tile, lane & 15);
    const int k0 = 32 * s + 8 * (lane >> 4);
    uint16_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (row && k0 + e < a.K) ? row[k0 + e] : (uint16_t)0;
    uint4 o;
    o.x = v[0] | ((uint32_t)v[1] << 16);
    o.y = v[2] | ((uint32_t)v[3] << 16);
    o.z = v[4] | ((uint32_t)v[5] << 16);
    o.w = v[6] | ((uint32_t)v[7] << 16);
    ((uint4 *)a.dst)[i] = o;
  }
}

// ---------------------------------------------------------------------------
// embedding + tree metadata + RoPE table
// ---------------------------------------------------------------------------

template <typename ET>
__device__ __forceinline__ float load_embed(const ET *e, size_t i);
template <>
__device__ __forceinline__ float load_embed<uint16_t>(const uint16_t *e, size_t i) {
  return bf2f(e[i]);
}
template <>
__device__ __forceinline__ float load_embed<float>(const float *e, size_t i) {
  return e[i];
}

// One workgroup per row.  bf16 models also get the first layer's RMSNorm here
// (a.gain set): the row is in registers anyway, so the norm costs no launch
// of its own (68M draft, one row: 3 us of 87).  Ancestors by pointer doubling
// over all rows at once, log2(n) rounds: following the parents one by one
// took 32 us for a 256-row chain, this kernel now takes 6.
template <typename ET>
__global__ __launch_bounds__(SB_MAX_ROWS) void k_embed_meta(EmbedArgs a, TreeArg tree) {
  const int t = blockIdx.x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __shared__ int16_t s_jump[SB_MAX_ROWS];
  __shared__ uint8_t s_on[SB_MAX_ROWS];  // row is on the path root..t
  __shared__ int s_cnt[SB_MAX_ROWS / 64];
  __shared__ float s_sq[SB_MAX_ROWS / 64];
  // the tree: a kernel argument (a dynamically indexed read is a memory access)
  int jump = (int)threadIdx.x < tree.n ? tree.parent[threadIdx.x] : -1;
  s_jump[threadIdx.x] = (int16_t)jump;
  s_on[threadIdx.x] = (int)threadIdx.x == t && t < tree.n;
  float *h = a.h + (size_t)t * a.hidden;
  float sq = 0.0f;
  constexpr int kMaxV = 8;
  float4 lo[kMaxV], hi[kMaxV];
  const bool vec = sizeof(ET) == 2 && (a.hidden & 7) == 0;
  if (t < a.n_tok) {
    int tok = a.tokens[t];
    tok = tok < 0 ? 0 : (tok >= a.vocab ? a.vocab - 1 : tok);  // ids are clamped
    const ET *e = (const ET *)a.embed + (size_t)tok * a.hidden;
    if (vec) {
      // bf16 rows: 8 elements per 16-byte load, every load of the row issued
      // before the first store (hidden <= 16384: at most 8 per thread)
      uint4 v[kMaxV];
      const int nv = a.hidden >> 3;
#pragma unroll
      for (int j = 0; j < kMaxV; ++j) {
        const int i = threadIdx.x + j * 256;
        if (i < nv) v[j] = ((const uint4 *)e)[i];
      }
#pragma unroll
      for (int j = 0; j < kMaxV; ++j) {
        const int i = threadIdx.x + j * 256;
        if (i < nv) {
          const uint32_t x[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
          lo[j].x = bf2f((uint16_t)(x[0] & 0xffff)); lo[j].y = bf2f((uint16_t)(x[0] >> 16));
          lo[j].z = bf2f((uint16_t)(x[1] & 0xffff)); lo[j].w = bf2f((uint16_t)(x[1] >> 16));
          hi[j].x = bf2f((uint16_t)(x[2] & 0xffff)); hi[j].y = bf2f((uint16_t)(x[2] >> 16));
          hi[j].z = bf2f((uint16_t)(x[3] & 0xffff)); hi[j].w = bf2f((uint16_t)(x[3] >> 16));
          ((float4 *)h)[2 * i] = lo[j];
          ((float4 *)h)[2 * i + 1] = hi[j];
          sq += (lo[j].x * lo[j].x + lo[j].y * lo[j].y) + (lo[j].z * lo[j].z + lo[j].w * lo[j].w) +
                (hi[j].x * hi[j].x + hi[j].y * hi[j].y) + (hi[j].z * hi[j].z + hi[j].w * hi[j].w);
        }
      }
    } else {
      for (int k = threadIdx.x; k < a.hidden; k += blockDim.x) h[k] = load_embed<ET>(e, k);
    }
  } else {
    for (int k = threadIdx.x; k < a.hidden; k += blockDim.x) h[k] = 0.0f;
  }
  __syncthreads();
  // round r: every row on the path marks its 2^r-th ancestor, then all jumps
  // double.  A mark seen within its own round only adds true ancestors.
  for (int step = 1; step < tree.n; step <<= 1) {
    const int next = jump >= 0 ? s_jump[jump] : -1;
    if (jump >= 0 && s_on[threadIdx.x]) s_on[jump] = 1;
    __syncthreads();
    jump = next;
    s_jump[threadIdx.x] = (int16_t)next;
    __syncthreads();
  }
  const unsigned long long on = __ballot(s_on[threadIdx.x] != 0);
  if (lane < 2) a.meta->anc[t][2 * w + lane] = (uint32_t)(on >> (32 * lane));
  if (lane == 0) s_cnt[w] = __popcll(on);
  if (sizeof(ET) == 2 && a.gain) {
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if (lane == 0) s_sq[w] = sq;
  }
  __syncthreads();
  const int rows = (s_cnt[0] + s_cnt[1]) + (s_cnt[2] + s_cnt[3]);
  const int pos = a.kv_len + (rows > 0 ? rows - 1 : 0);
  if (threadIdx.x == 0) a.meta->pos[t] = pos;
  if (a.rope && t < a.n_tok) {
    const int half = a.head_dim / 2;
    for (int j = threadIdx.x; j < half; j += blockDim.x) {
      const double ang = (double)pos * a.theta[j];
      double sn, cs;
      sincos(ang, &sn, &cs);
      a.rope[t * half + j] = make_float2((float)cs, (float)sn);
    }
  }
  // the first layer's norm in factored form, as k_rmsnorm_pack writes it
  if (sizeof(ET) == 2 && a.gain) {
    const int gbytes = a.hidden * 4;
    const __amdgpu_buffer_rsrc_t grs =
        __builtin_amdgcn_make_buffer_rsrc((void *)a.gain, 0, gbytes, kBufferDword3);
    f32x4 gv[kMaxV][2];
#pragma unroll
    for (int j = 0; j < kMaxV; ++j)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
        gv[j][hh] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                  grs, (threadIdx.x + j * 256) * 32 + hh * 16, 0, 0));
    const float mean = ((s_sq[0] + s_sq[1]) + (s_sq[2] + s_sq[3])) / (float)a.hidden;
    if (threadIdx.x == 0) a.rs[t] = t < a.n_tok ? 1.0f / sqrtf(mean + a.eps) : 0.0f;
#pragma unroll
    for (int j = 0; j < kMaxV; ++j) {
      const int i = threadIdx.x + j * 256;
      if (i >= a.xa_ks * 4) break;
      uint4 o = make_uint4(0, 0, 0, 0);  // columns past the width, rows past the tree
      if (t < a.n_tok && i * 8 < a.hidden) {
        o.x = f2bf(lo[j].x * gv[j][0][0]) | ((uint32_t)f2bf(lo[j].y * gv[j][0][1]) << 16);
        o.y = f2bf(lo[j].z * gv[j][0][2]) | ((uint32_t)f2bf(lo[j].w * gv[j][0][3]) << 16);
        o.z = f2bf(hi[j].x * gv[j][1][0]) | ((uint32_t)f2bf(hi[j].y * gv[j][1][1]) << 16);
        o.w = f2bf(hi[j].z * gv[j][1][2]) | ((uint32_t)f2bf(hi[j].w * gv[j][1][3]) << 16);
      }
      *(uint4 *)(a.xa + packed_index(t, i * 8, a.xa_ks)) = o;
    }
  }
}

// ---------------------------------------------------------------------------
// RMSNorm of the fp32 residual rows into the packed bf16 operand layout
// ---------------------------------------------------------------------------

// Threads per row of the RMSNorm kernel.
constexpr int kNormThreads = 512;

// One workgroup per row; a thread holds IPT groups of 8 columns in registers
// (one read of the row), the sum of squares is reduced across the block, and
// each group is written as one 16-byte store.
// With delta set, the n_delta slices of the previous projection (one per K
// range of a split-K GEMM, [n_delta][n_tok][hidden]) are first summed in
// slice order and added to the residual row, which is written back.
//
// The norm is applied in factored form, RMSNorm(h) g W^T = r (h g) W^T: the
// packed output is bf16(h g), and r = 1/sqrt(mean(h^2) + eps) goes to
// rs[t] for the projection's epilogue to multiply by.
//
// tap (H-RAD features, nullable): with tap_normed == 0 the residual row
// after the delta slices are added; with tap_normed != 0 the normalised row
// (h r) g in float32 (the last layer's state as the final norm leaves it).
//
// Every load of a thread (residual, all kMaxSplit delta slices, gains) is a
// buffer load issued before the first use, so a row costs one memory round
// trip; slices past n_delta, columns past hidden and rows past n_tok read
// zero (out-of-range offsets).
template <int IPT>
__global__ __launch_bounds__(kNormThreads) void k_rmsnorm_pack(float *__restrict__ h,
                                                               const float *__restrict__ delta,
                                                               int n_delta,
                                                               const float *__restrict__ g,
                                                               int hidden, int ks, int n_tok,
                                                               float eps,
                                                               uint16_t *__restrict__ out,
                                                               float *__restrict__ rs,
                                                               float *__restrict__ tap,
                                                               int tap_normed) {
  const int t = blockIdx.x;
  __shared__ float red[kNormThreads / 64];
  const int items = ks * 4;
  const bool live = t < n_tok;
  const int row_bytes = hidden * 4;
  const __amdgpu_buffer_rsrc_t hrs = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(h + (size_t)(live ? t : 0) * hidden), 0, live ? row_bytes : 0, kBufferDword3);
  const int dbytes = delta ? n_delta * n_tok * row_bytes : 0;
  const __amdgpu_buffer_rsrc_t drs =
      __builtin_amdgcn_make_buffer_rsrc((void *)(delta ? delta : h), 0, dbytes, kBufferDword3);
  const __amdgpu_buffer_rsrc_t grs =
      __builtin_amdgcn_make_buffer_rsrc((void *)g, 0, row_bytes, kBufferDword3);
  f32x4 hv[IPT][2], dv[IPT][kMaxSplit][2], gv[IPT][2];
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int k0 = (threadIdx.x + j * kNormThreads) * 8;
    const int vo = k0 < hidden ? k0 * 4 : row_bytes;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      hv[j][hh] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(hrs, vo, hh * 16, 0));
      gv[j][hh] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(grs, vo, hh * 16, 0));
    }
#pragma unroll
    for (int sl = 0; sl < kMaxSplit; ++sl) {
      const int dvo = (k0 < hidden && live) ? ((sl * n_tok + t) * hidden + k0) * 4 : dbytes;
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
        dv[j][sl][hh] =
            __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(drs, dvo, hh * 16, 0));
    }
  }
  float ss = 0.0f;
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int k0 = (threadIdx.x + j * kNormThreads) * 8;
    if (delta) {  // residual add of the previous projection, slices in order
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        f32x4 d = dv[j][0][hh];
#pragma unroll
        for (int sl = 1; sl < kMaxSplit; ++sl) d += dv[j][sl][hh];  // missing slices read 0
        hv[j][hh] += d;
      }
      if (live && k0 < hidden) {
        f32x4 *dst = (f32x4 *)(h + (size_t)t * hidden + k0);
        dst[0] = hv[j][0];
        dst[1] = hv[j][1];
        if (tap && !tap_normed) {  // the residual after the previous layer, for H-RAD
          f32x4 *tp = (f32x4 *)(tap + (size_t)t * hidden + k0);
          tp[0] = hv[j][0];
          tp[1] = hv[j][1];
        }
      }
    }
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int e = 0; e < 4; ++e) ss += hv[j][hh][e] * hv[j][hh][e];
  }
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = red[0];
#pragma unroll
  for (int i = 1; i < kNormThreads / 64; ++i) ss += red[i];
  const float scale = live ? 1.0f / sqrtf(ss / (float)hidden + eps) : 0.0f;
  if (rs && threadIdx.x == 0) rs[t] = scale;  // padding rows get 0
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int it = threadIdx.x + j * kNormThreads;
    if (it >= items) continue;
    const int k0 = it * 8;
    // columns past hidden have zero residual and gain: they pack to zero
    uint16_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = f2bf(hv[j][e >> 2][e & 3] * gv[j][e >> 2][e & 3]);
    uint4 o;
    o.x = v[0] | ((uint32_t)v[1] << 16);
    o.y = v[2] | ((uint32_t)v[3] << 16);
    o.z = v[4] | ((uint32_t)v[5] << 16);
    o.w = v[6] | ((uint32_t)v[7] << 16);
    *(uint4 *)(out + packed_index(t, k0, ks)) = o;
    if (tap && tap_normed && live && k0 < hidden) {  // the final norm's output, float32
      f32x4 *tp = (f32x4 *)(tap + (size_t)t * hidden + k0);
      tp[0] = (hv[j][0] * scale) * gv[j][0];
      tp[1] = (hv[j][1] * scale) * gv[j][1];
    }
  }
}

}  // namespace

hipError_t launch_pack_bf16(int kind, const sb_model_config &c, const void *src0, const void *src1,
                            const void *src2, void *dst, hipStream_t s) {
  PackArgs a;
  a.src0 = (const uint16_t *)src0;
  a.src1 = (const uint16_t *)src1;
  a.src2 = (const uint16_t *)src2;
  a.dst = (uint16_t *)dst;
  a.kind = kind;
  a.n_heads = c.n_heads;
  a.n_kv = c.n_kv_heads;
  a.head_dim = c.head_dim;
  a.ffn = c.ffn;
  const PackGeom g = pack_geom(c, kind);
  a.K = g.K;
  a.ks = g.ks;
  a.tiles = g.tiles;
  a.rows0 = g.rows;
  const size_t total = (size_t)a.tiles * a.ks * 64;
  size_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_pack, dim3((unsigned)blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_embed_meta(const EmbedArgs &a, const TreeArg &tree, int blocks, int bf16,
                             hipStream_t s) {
  if (bf16)
    hipLaunchKernelGGL(k_embed_meta<uint16_t>, dim3(blocks), dim3(SB_MAX_ROWS), 0, s, a, tree);
  else
    hipLaunchKernelGGL(k_embed_meta<float>, dim3(blocks), dim3(SB_MAX_ROWS), 0, s, a, tree);
  return hipGetLastError();
}

hipError_t launch_rmsnorm_pack(float *h, const float *delta, int n_delta, const float *g,
                               int hidden, int ks, int n_tok, int n_pad, float eps, uint16_t *out,
                               float *rs, hipStream_t s, float *tap, int tap_normed) {
  if (hidden % 8 != 0 || n_delta < 1 || n_delta > kMaxSplit) return hipErrorInvalidValue;
  const int ipt = (ks * 4 + kNormThreads - 1) / kNormThreads;
  switch (ipt) {
#define SB_IPT(n)                                                                              \
  case n:                                                                                      \
    hipLaunchKernelGGL(k_rmsnorm_pack<n>, dim3(n_pad), dim3(kNormThreads), 0, s, h, delta,        \
                       n_delta, g, hidden, ks, n_tok, eps, out, rs, tap, tap_normed);          \
    break;
    SB_IPT(1) SB_IPT(2) SB_IPT(3) SB_IPT(4) SB_IPT(5) SB_IPT(6) SB_IPT(7) SB_IPT(8)
#undef SB_IPT
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace sb
