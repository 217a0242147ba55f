// santa_dense.h -- the exact dense step (k_dense_stream and k_fused_dense; see
// santa_fused.h) and the S2ANTA-flash step on k_fused_dense.
#pragma once

#include "santa_fused.h"

namespace santa {

// ---------------------------------------------------------------------------
// S2ANTA-flash value stage (Sec. 3.3; App. "S2ANTA-Flash Pseudocode", Kernel 1)
// ---------------------------------------------------------------------------
// Flash draws of one split (Kernel 1): every tile tau of the split and every
// head h takes S_tile systematic draws on the tile's own distribution: draw i
// is the key whose tile-CDF interval holds ((i + a)/S_tile) l_tau, a = u of
// (head, tile) (App. A's inverse CDF, clamped to the tile).  Counts go to cnt;
// then each drawn key's count becomes the weight count * exp2(m_tau - m_w) *
// l_tau / S_tile (m_w: the split max), so the split's partial sum is
// o_w = sum_tau exp2(m_tau - m_w) l_tau O_tau with O_tau the tile estimate.
// Returns (block-uniform) whether any key was drawn.
template <int G>
__device__ __forceinline__ bool flash_draws(const FusedArgs &a, const float *P, int pitch, int *cnt,
                                            const float *tst, const float *mh, int start,
                                            int nrows, int64_t row0) {
  const int tid = threadIdx.x, tl2 = a.tile_log2, St = a.S_tile;
  const int ntile = (nrows + (1 << tl2) - 1) >> tl2;
  const int per_h = ntile * St;
  const float invSt = 1.0f / (float)St;
  const int gt0 = start >> tl2;  // global index of the split's first tile
  for (int i = tid; i < G * per_h; i += kThreads) {
    const int h = i / per_h, rem = i - h * per_h, tau = rem / St, is = rem - tau * St;
    const int t0 = tau << tl2, n = min(1 << tl2, nrows - t0);
    const float l = tst[(2 * h + 1) * (kSplitMax / 16) + tau];
    const float ua = a.u[(row0 + h) * a.Tmax + gt0 + tau];
    const float x = (((float)is + ua) * invSt) * l;
    const int k = lds_count_le(P + h * pitch + t0, n, x);
    const int j = t0 + (k < n ? k : n - 1);
    atomicAdd(&cnt[h * pitch + j], 1);
    if (a.idx_out) a.idx_out[((row0 + h) * a.Tmax + gt0 + tau) * St + is] = start + j;
  }
  __syncthreads();
  // counts -> weights
  for (int i = tid; i < G * nrows; i += kThreads) {
    const int h = i / nrows, j = i - h * nrows;
    const int c = cnt[h * pitch + j];
    if (c) {
      const int tau = j >> tl2;
      const float m = tst[(2 * h) * (kSplitMax / 16) + tau];
      const float l = tst[(2 * h + 1) * (kSplitMax / 16) + tau];
      cnt[h * pitch + j] = __float_as_int((float)c * (fast_exp2(m - mh[h]) * l * invSt));
    }
  }
  __syncthreads();
  return G * per_h > 0;
}

// ---------------------------------------------------------------------------
// Dense step
// ---------------------------------------------------------------------------
// PERSIST: a resident grid of R whole rows per round (small batches; the last
// min(G, Tb) arrivals of a row merge one head each).  Otherwise one work item
// per workgroup, hardware-scheduled (large batches): the row's last arrival
// merges every head and nothing waits, so the grid need not be resident.
// FLASH: the split's value stage is S2ANTA-flash (Sec. 3.3; App. "S2ANTA-Flash
// Pseudocode"): S_tile draws per tile and head on the tile's own distribution
// instead of the exact weighted sum; the split publishes o_w = sum_tau
// exp2(m_tau - m_w) l_tau O_tau with l_w = sum_tau exp2(m_tau - m_w) l_tau, so
// the same merge gives O = sum_tau W_tau O_tau / sum_tau W_tau (Kernel 2).
template <typename E, int G, bool PAGED, bool PERSIST, bool FLASH = false, bool APPEND = false>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(PERSIST ? 2 : 3))) void k_fused_dense(FusedArgs a) {
  // dynamic LDS: s [G][pitch] scores / weights, red [4][G*128] (also the merge scratch);
  // flash: s, cnt [G][pitch] (later red), list [pitch], tile statistics [G][2][kSplitMax/16]
  extern __shared__ __attribute__((aligned(16))) float dyn[];
  constexpr int pitch = kSplitMax;
  float *s = dyn;
  float *red = s + G * pitch;
  int *cnt = reinterpret_cast<int *>(red);
  int *list = cnt + imax(G * pitch, imax(4 * G * kHeadDim, a.T + kThreads));
  float *tst = reinterpret_cast<float *>(list + pitch);
  __shared__ float mh[G], lh[G], mtmp[4 * G], den;
  __shared__ int rank_lds;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = tid & 15;
  const int nrk = a.B * a.Hkv, T = a.T;
  const int R = gridDim.x / T;  // rows per round
  int rho, t;
  map_item(blockIdx.x, T, R, rho, t);
  QE<E> *out = static_cast<QE<E> *>(a.out);
  const int align = FLASH ? imax(kAlign, 1 << a.tile_log2) : kAlign;

  for (int rbase = 0; rbase < nrk; rbase += R) {
    __builtin_amdgcn_s_setprio(0);
    const int rowkv = rbase + rho;
    if (rowkv >= nrk) break;
    const int b = rowkv / a.Hkv, kvh = rowkv % a.Hkv;
    const int64_t row0 = (int64_t)b * a.Hq + kvh * G;
    const int L = seq_len(a.kv, b);
    int Ls, Tb;
    split_geometry(L, T, Ls, Tb, align);
    if constexpr (FLASH) {
      // tiles no split covers (past the row's length) have no draws
      if (a.idx_out && (t == Tb - 1 || (Tb == 0 && t == 0))) {
        const int t_end = (L + (1 << a.tile_log2) - 1) >> a.tile_log2;
        const int nt = (a.Tmax - t_end) * a.S_tile;
        for (int i = tid; i < G * nt; i += kThreads) {
          const int h = i / nt, k = i - h * nt;
          a.idx_out[((row0 + h) * a.Tmax + t_end) * a.S_tile + k] = -1;
        }
      }
    }
    if (t >= Tb) {
      if (Tb == 0 && t == 0)
        for (int o = tid; o < G * kHeadDim; o += kThreads) store_out(out + row0 * kHeadDim + o, 0.0f);
      continue;
    }
    const int start = t * Ls, nrows = min(Ls, L - start);
    if constexpr (APPEND) append_current<E, PAGED>(a.kv, b, kvh, a.Hkv, start, nrows, L);
    unsigned long long *sync = a.sync + (int64_t)rowkv * (kSyncStride / 2);
    const unsigned long long base =
        __hip_atomic_load(sync + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    float *part_row = a.part + (int64_t)rowkv * T * G * kHeadDim;

    const QRegs<E, G> qr = load_q<E, G>(static_cast<const QE<E> *>(a.q), b, a.Hq, kvh, c);
    const float2 sc = kv_scales<E>(a.kv, b, kvh, a.Hkv);  // FP8 cache: K and V scales
    float mx[G];
    constexpr int U = PERSIST ? score_unroll<E, G>() : (sizeof(E) == 1 && G <= 4 ? 8 : 4);
    score_tile<E, G, PAGED, U>(a.kv, b, kvh, start, nrows, qr, a.scale_log2 * sc.x, s, pitch, mx);
    block_max_heads<G>(mx, mtmp, mh);
    if constexpr (FLASH) {
      // tile CDFs (wave h: head h), the split normaliser l_w, zeroed counts
      constexpr int TS = kSplitMax / 16;
      for (int h = wave; h < G; h += kThreads / 64) {
        wave_tile_cdf(s + h * pitch, nrows, lane, a.tile_log2, tst + 2 * h * TS, tst + (2 * h + 1) * TS);
        const int ntile = (nrows + (1 << a.tile_log2) - 1) >> a.tile_log2;
        float l = 0.0f;
        for (int tau = lane; tau < ntile; tau += 64)
          l += fast_exp2(tst[2 * h * TS + tau] - mh[h]) * tst[(2 * h + 1) * TS + tau];
        l = wave_sum(l);
        if (lane == 0) lh[h] = l;
      }
      for (int i = tid; i < G * pitch; i += kThreads) cnt[i] = 0;
      __syncthreads();
      __builtin_amdgcn_s_setprio(3);
      const bool has = flash_draws<G>(a, s, pitch, cnt, tst, mh, start, nrows, row0);
      // the draws of a split can reach many distinct rows, so all 16 row slots
      // of the workgroup share the union list (8 rows in flight per slot, 4
      // for the wider accumulators of fp32 rows or G = 8)
      if (has) {
        constexpr int UG = (sizeof(E) <= 2 && G <= 4) ? 8 : 4;
        gather_union<E, G, PAGED, true, true, UG>(a.kv, b, kvh, start, nrows, s, pitch, cnt, list,
                                                  part_row + (int64_t)t * G * kHeadDim);
      } else {
        float2 *pz = reinterpret_cast<float2 *>(part_row + (int64_t)t * G * kHeadDim);
        for (int o2 = tid; o2 < G * kHeadDim / 2; o2 += kThreads) st_coherent(pz + o2, make_float2(0.f, 0.f));
      }
    } else {
      for (int h = wave; h < G; h += kThreads / 64) {
        float *sh = s + h * pitch;
        const float m = mh[h];
        float l = 0.0f;
        for (int j = lane; j < nrows; j += 64) {
          const float e = fast_exp2(sh[j] - m);
          sh[j] = e;
          l += e;
        }
        l = wave_sum(l);
        if (lane == 0) lh[h] = l;
      }
      __syncthreads();
      float acc[G][8];
      value_tile<E, G, PAGED, U>(a.kv, b, kvh, start, nrows, s, pitch, acc);
      __builtin_amdgcn_s_setprio(3);  // the merge chain issues ahead of streaming waves
      reduce_slots<G>(acc, red);
      float2 *mypart = reinterpret_cast<float2 *>(part_row + (int64_t)t * G * kHeadDim);
      for (int o2 = tid; o2 < G * kHeadDim / 2; o2 += kThreads) {
        float2 v = make_float2(0.0f, 0.0f);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          v.x += red[w * G * kHeadDim + 2 * o2];
          v.y += red[w * G * kHeadDim + 2 * o2 + 1];
        }
        st_coherent(mypart + o2, v);
      }
    }
    if (tid < G) st_coherent(a.stats + (row0 + tid) * T + t, make_float2(mh[tid], lh[tid]));

    // arrive; the last W arrivals merge one or more heads each
    const int W = PERSIST ? min(G, Tb) : 1;
    const int rank = row_arrive(sync, base, &rank_lds);
    if (rank < Tb - W) continue;
    if (rank == Tb - 1) {
      if (tid == 0)
        __hip_atomic_store(sync + 1, base + (unsigned long long)Tb, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    } else {
      row_wait(sync, base + (unsigned long long)Tb, a.err);
    }
    for (int h = rank - (Tb - W); h < G; h += W) {
      // a_t = exp2(m_t - m*) and the denominator sum_t a_t l_t
      float *al = red + kThreads;
      if (wave == 0) {
        const float2 *st = a.stats + (row0 + h) * T;
        float m = -kInf;
        for (int tt = lane; tt < Tb; tt += 64) m = fmaxf(m, ld_coherent(st + tt).x);
        m = wave_max(m);
        float d = 0.0f;
        for (int tt = lane; tt < Tb; tt += 64) {
          const float2 v = ld_coherent(st + tt);
          const float aa = fast_exp2(v.x - m);
          al[tt] = aa;
          d = fmaf(aa, v.y, d);
        }
        d = wave_sum(d);
        if (lane == 0) den = d;
      }
      __syncthreads();
      merge_head<QE<E>, G>(part_row, h, Tb, al, &den, sc.y, red, out + (row0 + h) * kHeadDim);
    }
  }
}

// ---------------------------------------------------------------------------
// Dense step of 16-bit and FP8 caches
// ---------------------------------------------------------------------------
// Lane `src` of every 16-lane row, on all lanes of the row.
template <int SRC>
__device__ __forceinline__ float row_bcast(float v) {
  return dpp<0x150 + SRC>(v);
}

// Online softmax state of one wave: running maximum of head lane % 16 (log2
// units), the lane's share of its sum, and the weighted V rows of the lane's
// row slot (lane / 16), 8 columns of every head.
template <int G>
struct WaveSoftmax {
  float m, l, acc[G][8];
};

// One tile of a wave: scores y (KeyRing::scores), then O += P V over the tile's
// rows.  Lane (slot, c) adds rows 4 slot .. + 3, whose weights the lanes of its
// own 16-lane row hold (head h in lane h): a row broadcast, no exchange
// through LDS.  PART: only the first `left` keys count.
template <typename E, int G, bool PART, typename R>
__device__ __forceinline__ void dense_tile(const R &kr, mf32x4 y, int vslot, int left, WaveSoftmax<G> &w) {
  const int lane = threadIdx.x & 63, r0 = 4 * (lane >> 4);
  if constexpr (PART) {
#pragma unroll
    for (int n = 0; n < 4; ++n) y[n] = r0 + n < left ? y[n] : -kInf;
  }
  const float tm = xor32_max(xor16_max(fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3]))));
  const float mn = fmaxf(w.m, tm);
  const float ms = mn == -kInf ? 0.0f : mn;  // no finite score yet: every weight is 0
  if (__any((lane & 15) < G && mn > w.m)) {
    const float f = fast_exp2(w.m - ms);
    w.l *= f;
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float fh = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), h));
#pragma unroll
      for (int i = 0; i < 8; ++i) w.acc[h][i] *= fh;
    }
    w.m = mn;
  }
  float p[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) p[n] = fast_exp2(y[n] - ms);
  w.l += (p[0] + p[1]) + (p[2] + p[3]);
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    float f[8];
    kr.row_chunk(r0 + n, vslot).to_float(f);
    if constexpr (PART) {
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = r0 + n < left ? f[i] : 0.0f;
    }
    auto head = [&](auto hc) {
      constexpr int h = decltype(hc)::value;
      if constexpr (h < G) {
        const float pw = row_bcast<h>(p[n]);
#pragma unroll
        for (int i = 0; i < 8; ++i) w.acc[h][i] = fmaf(pw, f[i], w.acc[h][i]);
      }
    };
    head(std::integral_constant<int, 0>{});
    head(std::integral_constant<int, 1>{});
    head(std::integral_constant<int, 2>{});
    head(std::integral_constant<int, 3>{});
    head(std::integral_constant<int, 4>{});
    head(std::integral_constant<int, 5>{});
    head(std::integral_constant<int, 6>{});
    head(std::integral_constant<int, 7>{});
  }
}

// Pairs of tiles (16 keys, their 16 value rows) in a wave's ring: two, 64 KB
// per workgroup (FP8: four of half the size), so two workgroups per CU.
template <typename E>
constexpr int dense_pairs() {
  return sizeof(E) == 1 ? 4 : 2;
}
template <typename E>
constexpr size_t dense_lds_bytes(int G, int T) {
  const size_t ring = ring_bytes<E>(2 * dense_pairs<E>());
  const size_t red = (size_t)4 * G * kHeadDim * 4, mrg = (size_t)G * T * 4;
  return ring > red ? (ring > mrg ? ring : mrg) : (red > mrg ? red : mrg);
}

// The exact step (Sec. 2, SDPA equation), one workgroup per (row, split).  It is
// bound by HBM: every key and value row is read once.  Each wave streams key and
// value tiles in turn through its own ring in LDS (KeyRing) and keeps its own
// online softmax, so nothing is exchanged and no barrier stands inside the
// stream, and the value rows of a tile are in flight while its keys are
// scored; the four waves are joined once at the end.  The split publishes o_t
// = sum exp2(s - m_t) V and (m_t, l_t); the row's last arrival merges O =
// sum_t a_t o_t / sum_t a_t l_t, a_t = exp2(m_t - m*).  24 ragged
// paged sequences of 512 to 16384 keys with the append: 207.2 (k_fused_dense,
// whose append variant spills) -> 163.4 us (4.5 -> 5.7 TB/s).  At 170 us, with a
// row's splits in a run, it took 164 us without the V arithmetic, 162 without
// the merge and 241 with rings of three pairs: more than about 64 KB per CU in
// flight only queues up.
template <typename E, int G, bool PAGED, bool APPEND = false>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_dense_stream(FusedArgs a) {
  extern __shared__ __attribute__((aligned(16))) float dyn[];
  constexpr int NP = dense_pairs<E>(), NB = 2 * NP;
  __shared__ float wm[4][G], wl[4][G], mh[G], lh[G], den[G];
  __shared__ int rank_lds;
  const int T = a.T, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Split-major, each split's rows turned by one: the splits that hold keys
  // come first, whatever share of the cache's capacity the rows fill, and a
  // row's splits alternate over the XCDs (workgroup w runs on XCD w % 8).
  // With the splits of a row in a run and T a multiple of 8, the first splits
  // of short rows all ran on the same few XCDs (batch 16 of 500 keys in a
  // cache of 32768: 126 us, so 16; of 8000: 138, so 90); full rows gain by the
  // heads of a token read together (batch 16 at 32k keys: 346 -> 328).
  const int nrk = a.B * a.Hkv, t = blockIdx.x / nrk, rowkv = (blockIdx.x % nrk + t) % nrk;
  const int b = rowkv / a.Hkv, kvh = rowkv % a.Hkv;
  const int64_t row0 = (int64_t)b * a.Hq + kvh * G;
  QE<E> *out = static_cast<QE<E> *>(a.out);
  const int L = seq_len(a.kv, b);
  int Ls, Tb;
  split_geometry(L, T, Ls, Tb);
  if (Ls < a.Ls) {  // short rows: not T tiny splits, but as many as fill the chip
    Ls = max(Ls, min(a.Ls, (((L + a.fill - 1) / a.fill) + kAlign - 1) & ~(kAlign - 1)));
    Tb = (L + Ls - 1) / Ls;
  }
  if (t >= Tb) {
    if (Tb == 0 && t == 0)  // empty sequence: zero output
      for (int o = tid; o < G * kHeadDim; o += kThreads) store_out(out + row0 * kHeadDim + o, 0.0f);
    return;
  }
  const int start = t * Ls, nrows = min(Ls, L - start);
  if constexpr (APPEND) append_current<E, PAGED>(a.kv, b, kvh, a.Hkv, start, nrows, L);

  WaveSoftmax<G> w;
  w.m = -kInf;
  w.l = 0.0f;
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int i = 0; i < 8; ++i) w.acc[h][i] = 0.0f;
  const float2 sc = kv_scales<E>(a.kv, b, kvh, a.Hkv);  // FP8 cache: K and V scales
  {
    const QFrag qf = load_q_frag<E, G>(static_cast<const QE<E> *>(a.q), row0);
    const float scale = a.scale_log2 * sc.x;
    KeyRing<E, G, PAGED, NB> kr(a.kv, wave, reinterpret_cast<char *>(dyn));
    const int mine = kr.item(b, start, nrows, page_window<PAGED>(a.kv, b, start, nrows));
    constexpr int NL = KeyRing<E, G, PAGED, NB>::NL;
    auto copy = [&](int i, int pair) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the pair's last reads are done
      kr.copy(a.kv.k, kvh, i, 2 * pair);
      kr.copy(a.kv.v, kvh, i, 2 * pair + 1);
    };
#pragma unroll
    for (int i = 0; i < NP - 1; ++i)
      if (i < mine) copy(i, i);
    // the queries are complete, in the compiler's books too: it puts no wait
    // of its own into the stream
    __builtin_amdgcn_s_waitcnt(0);
    int pair = 0, ahead = NP - 1;
#pragma unroll 1
    for (int i = 0; i < mine; ++i) {
      const bool more = i + NP - 1 < mine;
      if (more) {
        copy(i + NP - 1, ahead);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((2 * NP - 1) * NL) : "memory");  // the keys have landed
      } else {
        wait_stores();
      }
      const mf32x4 y = kr.scores(qf, 2 * pair, scale);
      if (more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((2 * NP - 2) * NL) : "memory");  // the value rows too
      const int left = nrows - (wave + 4 * i) * kTileKeys;
      if (left >= kTileKeys) dense_tile<E, G, false>(kr, y, 2 * pair + 1, left, w);
      else dense_tile<E, G, true>(kr, y, 2 * pair + 1, left, w);
      pair = pair + 1 == NP ? 0 : pair + 1;
      ahead = ahead + 1 == NP ? 0 : ahead + 1;
    }
  }
  // join the four waves: m_t, l_t, then o_t in wave order
  const float l = xor32_sum(xor16_sum(w.l));
  if (lane < G) wm[wave][lane] = w.m, wl[wave][lane] = l;
  __syncthreads();
  if (tid < G) {
    const float m = fmaxf(fmaxf(wm[0][tid], wm[1][tid]), fmaxf(wm[2][tid], wm[3][tid]));
    const float ms = m == -kInf ? 0.0f : m;
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float f = fast_exp2(wm[i][tid] - ms);
      s = fmaf(f, wl[i][tid], s);
      wm[i][tid] = f;
    }
    mh[tid] = m;
    lh[tid] = s;
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float f = wm[wave][h];
#pragma unroll
    for (int i = 0; i < 8; ++i) w.acc[h][i] *= f;
  }
  float *red = dyn;  // the rings are done with
  reduce_slots<G>(w.acc, red);
  unsigned long long *sync = a.sync + (int64_t)rowkv * (kSyncStride / 2);
  const unsigned long long base = __hip_atomic_load(sync + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  float *part_row = a.part + (int64_t)rowkv * T * G * kHeadDim;
  float2 *mypart = reinterpret_cast<float2 *>(part_row + (int64_t)t * G * kHeadDim);
  for (int o2 = tid; o2 < G * kHeadDim / 2; o2 += kThreads) {
    float2 v = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v.x += red[i * G * kHeadDim + 2 * o2];
      v.y += red[i * G * kHeadDim + 2 * o2 + 1];
    }
    st_coherent(mypart + o2, v);
  }
  if (tid < G) st_coherent(a.stats + (row0 + tid) * T + t, make_float2(mh[tid], lh[tid]));

  const int rank = row_arrive(sync, base, &rank_lds);
  if (rank != Tb - 1) return;
  if (tid == 0)
    __hip_atomic_store(sync + 1, base + (unsigned long long)Tb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  float *al = dyn;  // [G][T]: a_t
  for (int h = wave; h < G; h += kThreads / 64) {
    const float2 *st = a.stats + (row0 + h) * T;
    constexpr int CH = kMaxSplits / 64;
    float2 v[CH];
    float m = -kInf, d = 0.0f;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      v[i] = lane + 64 * i < Tb ? ld_coherent(st + lane + 64 * i) : make_float2(-kInf, 0.0f);
      m = fmaxf(m, v[i].x);
    }
    m = wave_max(m);
#pragma unroll
    for (int i = 0; i < CH; ++i)
      if (lane + 64 * i < Tb) {
        const float at = fast_exp2(v[i].x - m);
        al[h * T + lane + 64 * i] = at;
        d = fmaf(at, v[i].y, d);
      }
    d = wave_sum(d);
    if (lane == 0) den[h] = d;
  }
  __syncthreads();
  for (int o2 = tid; o2 < G * kHeadDim / 2; o2 += kThreads) {  // column pairs; split order, 32 in flight
    const int o = 2 * o2, h = o / kHeadDim;
    float sx = 0.0f, sy = 0.0f;
    constexpr int NV = 32;
    for (int t0 = 0; t0 < Tb; t0 += NV) {
      float2 v[NV];
#pragma unroll
      for (int i = 0; i < NV; ++i)
        v[i] = t0 + i < Tb ? ld_coherent(reinterpret_cast<const float2 *>(part_row + (int64_t)(t0 + i) * G * kHeadDim + o))
                           : make_float2(0.0f, 0.0f);
#pragma unroll
      for (int i = 0; i < NV; ++i)
        if (t0 + i < Tb) {
          const float at = al[h * T + t0 + i];
          sx = fmaf(at, v[i].x, sx);
          sy = fmaf(at, v[i].y, sy);
        }
    }
    store_out(out + row0 * kHeadDim + o, sx * sc.y / den[h]);
    store_out(out + row0 * kHeadDim + o + 1, sy * sc.y / den[h]);
  }
}

template <typename E>
hipError_t launch_dense_e(const Plan &p, const KvView &kv, const void *q, float scale_log2,
                          void *out, char *ws, hipStream_t st) {
  FusedArgs args = make_args(p, kv, q, out, scale_log2, ws);
  return with_g_paged(p.G, kv.bt != nullptr, [&](auto gc, auto paged) -> hipError_t {
    constexpr int G = decltype(gc)::value;
    constexpr bool PG = decltype(paged)::value;
    constexpr bool AP = sizeof(E) > 1;  // an FP8 cache takes no append
    const bool ap = AP && kv.k_new != nullptr;
    const int rows = p.B * p.Hkv;
    const size_t lds = (size_t)fused_dense_floats(G, kSplitMax, p.T) * 4;
    const void *res = ap ? reinterpret_cast<const void *>(&k_fused_dense<E, G, PG, true, false, AP>)
                         : reinterpret_cast<const void *>(&k_fused_dense<E, G, PG, true>);
    // k_fused_dense beyond one resident round: float32, and the short rows
    // that dense_streams leaves to it
    constexpr bool many = sizeof(E) == 4 || G == 1 || (G == 2 && sizeof(E) == 1);
    auto resident = [&] { return rows * p.T <= capacity_of(res, lds); };
    if constexpr (sizeof(E) <= 2) {
      if (dense_streams(p, PG) || (!many && !resident())) {
        // Rows of fewer than 512 T keys take fewer splits than T, of up to 512
        // keys, but together at least two workgroups per CU if the row count
        // allows it.  Splits of 512 keys throughout left batch 2 of 500 keys
        // (capacity 65536) at 20 us for 8; one workgroup per CU is level or
        // better in full caches of short rows and 10 % behind on ragged ones (4
        // paged sequences of 500 to 9000 keys 21.6 us for 18.2).
        args.Ls = std::min(p.Ls, 512);
        args.fill = (512 + rows - 1) / rows;
        const void *fn = ap ? reinterpret_cast<const void *>(&k_dense_stream<E, G, PG, AP>)
                            : reinterpret_cast<const void *>(&k_dense_stream<E, G, PG>);
        void *params[] = {&args};
        const CallTimer tm = call_timer();
        return hipExtLaunchKernel(fn, dim3(rows * p.T), dim3(kThreads), params,
                                  dense_lds_bytes<E>(G, p.T), st, tm.start, tm.stop, 0);
      }
    }
    if (resident()) return launch_resident(res, p, args, lds, st);
    if constexpr (many) {
      void *params[] = {&args};
      const CallTimer tm = call_timer();
      return hipExtLaunchKernel(ap ? reinterpret_cast<const void *>(&k_fused_dense<E, G, PG, false, false, AP>)
                                   : reinterpret_cast<const void *>(&k_fused_dense<E, G, PG, false>),
                                dim3(rows * p.T), dim3(kThreads), params, lds, st, tm.start, tm.stop, 0);
    }
    return hipErrorInvalidConfiguration;  // (not reached)
  });
}

template <typename E>
hipError_t launch_flash_e(const Plan &p, const KvView &kv, const void *q, float scale_log2,
                          int tile_log2, int S_tile, const float *u, int32_t *idx_out, void *out,
                          char *ws, hipStream_t st) {
  FusedArgs args = make_args(p, kv, q, out, scale_log2, ws);
  args.u = u;
  args.idx_out = idx_out;
  args.tile_log2 = tile_log2;
  args.S_tile = S_tile;
  args.Tmax = (p.n_k + (1 << tile_log2) - 1) >> tile_log2;
  return with_g_paged(p.G, kv.bt != nullptr, [&](auto gc, auto paged) -> hipError_t {
    constexpr int G = decltype(gc)::value;
    constexpr bool PG = decltype(paged)::value;
    const size_t lds = (size_t)fused_flash_floats(G, kSplitMax, p.T) * 4;
    constexpr bool AP = sizeof(E) > 1;  // an FP8 cache takes no append
    const bool ap = AP && kv.k_new != nullptr;
    const void *res = ap ? reinterpret_cast<const void *>(&k_fused_dense<E, G, PG, true, true, AP>)
                         : reinterpret_cast<const void *>(&k_fused_dense<E, G, PG, true, true>);
    const int rows = p.B * p.Hkv;
    if (rows * p.T <= capacity_of(res, lds))  // one resident round
      return launch_resident(res, p, args, lds, st);
    void *params[] = {&args};
    const CallTimer tm = call_timer();
    return hipExtLaunchKernel(ap ? reinterpret_cast<const void *>(&k_fused_dense<E, G, PG, false, true, AP>)
                                 : reinterpret_cast<const void *>(&k_fused_dense<E, G, PG, false, true>),
                              dim3(rows * p.T), dim3(kThreads), params, lds, st, tm.start, tm.stop,
                              0);
  });
}

}  // namespace santa
