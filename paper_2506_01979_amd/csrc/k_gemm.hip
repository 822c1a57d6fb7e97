// Launch planning and dispatch of the skinny matrix-core GEMM (the kernel
// is in sb_gemm_kernel.h, built once per epilogue kind in k_gemm_*.hip).
//
// The residual projections, about one tile per compute unit, split K across
// workgroups and leave partial deltas for the next RMSNorm (RESID), or run
// unsplit and apply the following RMSNorm themselves (RESID_NORM).
#include "sb_internal_fwd.h"

namespace sb {

namespace {

int device_cus() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      cus = 256;
  }
  return cus;
}

// Tiles per pass with a k_gemm kernel.
constexpr int kNTs[] = {1, 2, 3, 4, 6, 8};

}  // namespace

// Wide plan: the fewest token blocks of at most kWideTtCap tiles; the tile
// groups fill the compute units; a group's tiles go in as few passes over K
// as the accumulators allow.  The residual projections also split K over the
// S <= kMaxSplit workgroups that make the bytes a workgroup moves, passes
// (tiles + token tiles) / S, least (fewer slices on ties; 13B down at 129
// rows: S = 4 35 us, S = 2 48).
static GemmPlan plan_wide(int epi, int tiles, int ks, int tt_all, int cus) {
  GemmPlan p{};
  p.wide = 1;
  p.tblocks = (tt_all + kWideTtCap - 1) / kWideTtCap;
  p.tt = (tt_all + p.tblocks - 1) / p.tblocks;
  const int cap = kWidePairs / p.tt < kWideNtCap ? kWidePairs / p.tt : kWideNtCap;
  const int most = epi == EPI_RESID ? kMaxSplit : 1;
  long long best = 0;
  for (int S = 1; S <= most && (S == 1 || S * 4 <= ks); ++S) {
    int groups = cus / (p.tblocks * S);
    if (groups < 1) groups = 1;
    if (groups > tiles) groups = tiles;
    const int per_wg = (tiles + groups - 1) / groups;
    const int passes = (per_wg + cap - 1) / cap;
    int nt = (per_wg + passes - 1) / passes;
    if (nt < 2) nt = 2;
    const long long cost = 12LL * passes * (nt + p.tt) / S;  // 12: whole for every S
    if (S == 1 || cost < best) {
      best = cost;
      p.nt = nt;
      p.split = S;
      p.groups = groups;
    }
  }
  p.grid = p.tblocks * p.split * p.groups;
  return p;
}

GemmPlan plan_gemm(int epi, int tiles, int ks, int n_tok) {
  GemmPlan p{};
  const int nc = ks / 8;
  const int tt_all = (n_tok + 15) / 16;
  const int cus = device_cus();
  if (tt_all > kWideFrom) return plan_wide(epi, tiles, ks, tt_all, cus);
  p.tt = tt_all;
  p.tblocks = 1;
  // Projections that add into the residual stream have as many tiles as the
  // model is wide, about one per compute unit: they split K so that each
  // workgroup owns several tiles; the next RMSNorm sums the partial deltas.
  // Up to two tiles per unit, K is halved, or quartered where that leaves the
  // fullest workgroup less to do: at 320 tiles 5 quarters instead of 3 halves,
  // 13B's down projection 29.6 -> 27.8 us at 33 rows, 36.4 -> 30.6 at 64,
  // 25.8 -> 25.6 at 2; 512 tiles (70B) are 4 halves or 8 quarters, 71.6
  // against 74.2 us at 17 rows.
  const int per_cu = (tiles + cus - 1) / cus;
  auto most_of = [&](int s) {  // tiles of the fullest workgroup
    const int g = cus / s < 1 ? 1 : cus / s;
    return (tiles + g - 1) / g;
  };
  int S = 1;  // RESID_NORM: 1
  if (epi == EPI_RESID && per_cu <= 2)
    S = per_cu == 1 || most_of(kMaxSplit) * 2 < most_of(2) * kMaxSplit ? kMaxSplit : 2;
  if (S > nc) S = nc;
  if (S < 1) S = 1;
  int groups = cus / S;
  if (groups > tiles) groups = tiles;
  const int per_wg = (tiles + groups - 1) / groups;
  const int passes = (per_wg + kGemmNtCap - 1) / kGemmNtCap;
  const int need = (per_wg + passes - 1) / passes;
  for (int v : kNTs)
    if (v >= need) {
      p.nt = v;
      break;
    }
  p.split = S;
  p.groups = groups;
  p.grid = groups * S;
  return p;
}

bool resid_norm_fusable(int tiles, int ks, int n_tok, int *groups) {
  const GemmPlan p = plan_gemm(EPI_RESID_NORM, tiles, ks, n_tok);
  if (groups) *groups = p.groups;
  return n_tok <= kNormFuseRows && !p.wide && p.groups <= kSsGroups &&
         (tiles + p.groups - 1) / p.groups <= p.nt && p.nt * p.tt <= kRedPairs;
}

hipError_t launch_gemm(int epi, const GemmArgs &a, int tiles, int *split, hipStream_t s) {
  if (a.ks % 8 != 0 || a.n_tok <= 0 || a.n_tok > SB_MAX_ROWS) return hipErrorInvalidValue;
  if (epi == EPI_RESID_NORM && (!resid_norm_fusable(tiles, a.ks, a.n_tok, nullptr) || !a.gain ||
                                !a.xn || !a.ss || a.xn_ks * 32 < a.out_rows))
    return hipErrorInvalidValue;
  if (a.ss_in && (a.n_tok > kNormFuseRows || a.ss_groups < 1 || a.ss_groups > kSsGroups ||
                  epi == EPI_RESID_NORM || epi == EPI_QKV))
    return hipErrorInvalidValue;
  const GemmPlan p = plan_gemm(epi, tiles, a.ks, a.n_tok);
  // k_gemm_wide has no fused softmax statistics: the caller runs the
  // separate pass for such shapes
  if (p.wide && a.lm_part) return hipErrorInvalidValue;
  GemmArgs b = a;
  b.epi = epi;
  b.tiles = tiles;
  b.split = p.split;
  b.groups = p.groups;
  b.tblocks = p.tblocks;
  if (split) *split = p.split;
  switch (epi) {
    case EPI_QKV: return launch_gemm_qkv(b, p, s);
    case EPI_RESID: return launch_gemm_resid(b, p, s);
    case EPI_SWIGLU: return launch_gemm_swiglu(b, p, s);
    case EPI_LOGITS: return launch_gemm_logits(b, p, s);
    case EPI_RESID_NORM: return launch_gemm_resid_norm(b, p, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sb
