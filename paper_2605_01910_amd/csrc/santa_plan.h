// santa_plan.h -- internal definitions shared by the host dispatcher and the
// kernels of libsanta: the launch plan (split length, workspace carve-up) and
// the by-value views the kernels receive.  Not part of the public ABI.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace santa {

constexpr int kHeadDim = 128;   // supported head dimension
constexpr int kThreads = 256;   // threads per workgroup (4 waves of 64)
constexpr int kSplitMax = 1024; // largest KV split (keys) handled by one workgroup
constexpr int kMaxSplits = 256; // largest number of splits per row in the fused kernels
constexpr int kRowTMax = 64;    // largest number of splits per row of the scheduled sampled path
// Scheduled path: grids of at most this many workgroups (one per CU of the
// MI355X) wait at the row barrier by polling the statistics directly and
// may hold large threshold sets in LDS.
constexpr int kDirectPollMax = 256;
// Per KV row, the fused paths keep a sync block of kSyncStride ints: the
// counters in the first 256 bytes, then (at u64 index kMailOffset) the
// scheduled sampled path's statistics mailbox, one u64 per (head < 8, split <
// kRowTMax), zero whenever no call is running.
constexpr int kMailOffset = 32;
constexpr int kSyncStride = 2 * kMailOffset + 2 * 8 * kRowTMax;
constexpr int kSyncRowsMax = 4096; // KV rows (batch * kv heads) of the fused paths' counter area
constexpr int kErrBytes = 128;    // the error flag's section

// Per-call launch plan.  The KV sequence of every (batch, kv head) row is cut
// into T splits of Ls keys; each split is one workgroup.  All sizes below are
// a pure function of (shape, n_k, S, kind), so santa_workspace_size() and the
// decode calls agree on the layout.
struct Plan {
  int B, Hq, Hkv, G, dtype;
  int elem;     // element type of K and V: 0 bfloat16, 1 float32, 2 FP8 E4M3 (q, out bfloat16)
  int n_k;      // max context length
  int Ls;       // keys per split (multi-kernel: multiple of 16; fused: longest split of
                // any row, multiple of 64; <= kSplitMax)
  int T;        // splits per row for n_k keys
  int S;        // samples per row (0 for dense)
  int kind;     // santa_kind_t
  int fused;    // 1: single persistent launch (per-row split lengths), 0: multi-kernel
  int rows;     // fused systematic / stratified: 1 = one hardware-scheduled launch, a
                // workgroup per split with row barriers (k_row_sampled)
  int split2;   // fused sampled: 1 = stream + CDF stash, then one workgroup per
                // query head; 0 = one persistent launch
  int64_t npitch;  // two-launch sampled: stash entries per query head (n_k rounded up to 64)
  // workspace carve-up (byte offsets, 256-aligned)
  size_t off_stats;  // float2 [B*Hq*T]     per-split (max, sum) in log2 units
  size_t off_stash;  // float  [B*Hq*T*Ls] split-local CDF of each row (multi-kernel);
                     // uint16 [B*Hq*npitch] in-block CDF fraction of each key (two launches)
  size_t off_coarse; // float  [B*Hq*npitch/32] fused: CDF at every 32-key block end
  size_t off_offs;   // float  [B*Hq*(T+1)] global split offsets of the CDF
  size_t off_alpha;  // float  [B*Hq*T]     per-split rescale exp2(m_t - m*)
  size_t off_rowst;  // float2 [B*Hq]       (m*, Z) per row
  size_t off_part;   // float  [B*Hkv*T*G*128] per-split partial outputs
  size_t off_flag;   // int    [B*Hkv*T]    1 if the split holds samples
  size_t off_bw;     // float  [B*Hq*128]   Bernoulli query weights
  size_t off_blist;  // int    [B*Hkv*128]  Bernoulli feature list
  size_t off_bn;     // int    [B*Hkv]      Bernoulli feature count
  size_t off_err;    // int    [1]          fused: a wait gave up
  size_t off_sync;   // u64    [kSyncRowsMax*kSyncStride/2] fused: per-row sync blocks
                     // (counters, mailbox); the area has the same offset and size in every
                     // layout, so calls of any kind and shape find their counters where
                     // earlier calls left them
  size_t total;
};

// The dense step of 16-bit and FP8 caches takes k_dense_stream on grids (KV
// rows x splits) of several workgroups per CU, where its continuous stream
// counts (us, this kernel / k_fused_dense, 32k keys unless said): batch 4 95 /
// 110, batch 16 328 / 365 (G = 1 318 / 344, G = 8 356 / 437), head-major 333 /
// 344, FP8 211 / 237, groups of 8 at batch 4 107 / 147, 24 ragged paged
// sequences up to 16k 164 / 199; grids of 520 to 1024: batch 3 74.3 / 74.6, 5
// at 16k 64 / 69, 9 at 8k 56 / 65 (FP8 42 / 50).
// At two workgroups per CU a contiguous cache streams as fast through registers
// and the deeper rings only queue up (batch 1 34.7 / 30.4, batch 2 55.1 / 52.1,
// batch 8 at 8k 54.2 / 50.7); a paged one does not (4 ragged sequences up to
// 9000 keys 20 / 28) unless its splits are of 64 keys, one tile per wave:
// batch 1 of 4000 keys G = 2 13.1 / 13.7, G = 4 13.1 / 14.6, but G = 1 13.7 /
// 12.5 and G = 8 20.2 / 19.2.
// Rows in one split (more than 512 rows of up to 1024 keys) are too short for
// a stream where the arithmetic is little: batch 128, G = 1, contiguous, 64
// keys 13.1 / 11.9, 256 30.6 / 26.6, 400 37.8 / 38.4; FP8 64 12.0 / 11.0, 256
// 21.3 / 17.2, 1000 52.7 / 48.8 (G = 2 13.2 / 15.5, 23.4 / 21.5, 55.2 / 53.4);
// paged 16 keys 12.2 / 10.6 (FP8 64 12.5 / 12.7, batch 300 32.1 / 29.6).
inline bool dense_streams(const Plan &p, bool paged) {
  const int64_t grid = (int64_t)p.B * p.Hkv * p.T;
  if (p.elem == 1 || grid <= (paged ? 256 : 512)) return false;
  if (grid <= 512) return p.Ls > 64 || p.G == 2 || p.G == 4;
  if (p.T == 1 && p.G == 1) return p.Ls > (paged ? 64 : p.elem == 2 ? 1024 : 256);
  if (p.T == 1 && p.G == 2 && p.elem == 2 && !paged) return p.Ls <= 64;
  return true;
}

// The scheduled sampled step (k_row_sampled) scores on the matrix cores
// (ring_scores) in groups of eight and on paged 16-bit caches.  Its rings leave
// fewer workgroups per CU than the register form: 2 for 3 at G = 8, 3 (G = 1: 4)
// for 4 to 6 at smaller G.  Workgroups that wait at a row barrier or gather
// don't stream, so the smaller number shows where it takes a round more (us,
// ring_scores / score_tile, S = 128 to 256, full rows unless said):
// - G <= 4, paged: one resident round (G = 4, 32k keys: batch 1 18.5 / 25.0,
//   batch 3, 768 workgroups, 41.9 / 44.6; batch 4 61.5 / 55.7, 12 152 / 149;
//   16 sequences of 800 to 8000 keys 53 / 48, 300 of 500 206 / 149; G = 2 level
//   with that).  G = 1 also beyond two rounds, where the part of a round is
//   small (batch 4 50.8 / 52.0; 5, 1280 workgroups, 64.6 / 62.1, 24 of 8000 keys
//   73.0 / 71.3; 90 of 3000, 2160, 100.4 / 100.4, of 1500 to 3000 81 / 86, 60 of
//   8000 161 / 164).
// - G = 8: everywhere (batch 1 29.9 / 40.7, batch 16 279 / 296; paged 30.8 /
//   48.6, 297 / 352; FP8 27.7 / 41.2; 24 sequences of 3000 keys, 576 workgroups,
//   62 / 66, of 300 to 3000 39 / 55) but in rows of one or two splits, which
//   gather more than they stream, on grids that take a round more at two per CU
//   than at three (80 sequences of 500 keys, 640 workgroups: 64 / 54, paged 78 /
//   64, FP8 59 / 53; 128, 1024: 109 / 117; 300, 2400: 282 / 260; two splits: 36
//   of 2000 73 / 69, paged 83 / 80, 46 of 860 to 1090 and S = 877 152 / 116; but
//   FP8 64 / 70).
inline bool rows_ring(const Plan &p, bool paged) {
  const int64_t grid = (int64_t)p.B * p.Hkv * p.T;
  if (p.G == 1) return paged && p.elem == 0 && (grid <= 1024 || grid > 2048);
  if (p.G < 8) return paged && p.elem == 0 && grid <= 768;
  if (p.T == 1 || (p.T == 2 && p.elem == 0)) return (grid + 511) / 512 <= (grid + 767) / 768;
  return p.elem != 1;
}

// KV cache as the kernels see it (see santa_kv_t for the addressing rules).
struct KvView {
  const void *k, *v;
  int64_t sb, sn, sh;
  const int32_t *ctx;   // nullable
  const int32_t *bt;    // nullable (contiguous)
  int32_t ps_log2;      // log2(page_size)
  int32_t max_pages;
  int32_t n_k;
  const void *k_new, *v_new;  // nullable: the current token's rows [B, Hkv, 128], appended in-launch
  const float *ks, *vs;       // FP8 cache: dequantisation scales [B*Hkv] of K and V (else null)
};

struct KtView {
  const void *kt;
  int64_t sb, sh, sd;
};

}  // namespace santa
