// dK/dV work items of the SRA backward on gfx950 (the gradient is described in sra_bwd.hip).
//
// Key-major: a work item is a tile of 256 keys of one stream and head; its four waves (one per
// SIMD) own 64 keys each, as four 16-key MFMA blocks, and keep those keys' V, and the first 64
// head dims of K, in VGPRs and their dK and dV sums in AGPRs for the whole item. The other head
// dims of K (d = 128) sit in LDS: with all of K in registers the kernel does not fit, with all
// of it in LDS the query tiles do not. The query rows that see the keys stream through LDS in
// 64-row tiles, taken as two 32-row halves (gen keys: the gen queries of the sample; ref keys:
// the gen queries plus the ref queries of the key's group; a tile may hold keys of two groups,
// and then each group's query span reaches only its own range of the tile's keys):
//     S = Q K^T, dP = dO V^T, P = exp2(S scale log2e - LSE), dS = P (dP - D),
//     dV^T += dO^T P, dK^T += Q^T dS.
// Each Q and dO fragment read from LDS feeds all four key blocks of a wave. A half's dK product
// runs behind the next half's S product, so that it hides half of the exponentials (dP the
// others, dV the dS). Built with MFMAs in VGPR form (S and dP live in VGPRs); the dK/dV
// products are written as AGPR-accumulating MFMAs (mfma16_agpr). Bound by the clock that the board's
// power allows (720p: 2.20 of 2.4 GHz) and by issue: the MFMA pipes are busy 58 % of the cycles, with 1.3
// vector instructions per MFMA; waves wait for an issue slot in 29 % of their cycles, for data in 16 %.
// 480p, 5 heads 7.36 ms with 32x32x16 MFMAs in 32-query tiles, 6.69 ms so.
#pragma once
#include "sra_kernels.h"
#include "sra_tiles.h"

namespace sra {

constexpr int kDkvWaves = kDkvKeyTile / 64;  // one wave per SIMD, 64 keys each
constexpr int kDkvTile = 64;                 // queries per LDS tile
constexpr int kDkvBufs = 3;
constexpr int kDkvLook = 2;                  // LDS fragments are read this many groups of four MFMAs ahead
constexpr int kRegChunks = 2;                // 32-dim chunks of K held in registers

template <int D>
struct DkvState {
  static constexpr int NC = D / 32, ND = D / 16;
  bf16x8 vf[4][NC];          // V of the wave's four key blocks as B fragments (lane = key)
  bf16x8 kf[4][kRegChunks];  // K of head dims 0..63, likewise
  floatx4 dk[4][ND];         // dK^T accumulators (lane = key), 16 head dims each
  floatx4 dv[4][ND];         // dV^T accumulators
  bf16x8 ds[4];              // dS of the half before: B fragments (elements 0..3 are queries
                             // 4 g + i, 4..7 queries 16 + 4 g + i; g = lane / 16)
};

// LDS byte addresses of a wave's fragments: row fragments of c = 0 and transpose reads of db = 0
// of a tile at LDS address 0 (the others by XOR), and row fragments of the wave's K rows.
struct DkvAddr {
  uint32_t row, tr, k;
};

// One 32-query half for the wave's 64 keys: S, dK of the half before, dP, dV. qt, dt: LDS
// addresses of this half's Q and dO rows, stat: of its rows' LSE (log2 units; -D 256 bytes
// further), qtp: of the Q rows of the half before. S = Q K^T and dP = dO V^T have lanes = keys and
// registers = query rows, so P and dS are directly the B fragments of the products they enter.
// Each MFMA is followed by its share of the vector work (a 16x16x32 MFMA hides about 8 cycles of
// it) and a scheduling barrier; LDS fragments are read one group of four MFMAs ahead. Rows
// outside the span have LSE = +inf, so P = 0. kRange: the lane's key of block kb takes part only
// if bit kb of kv is set. hook(u) runs behind MFMA group u of the half's D / 4.
template <int D, bool kRange, class Hook>
__device__ __forceinline__ void dkv_half(DkvState<D>& st, const DkvAddr& ad, uint32_t qt, uint32_t dt, uint32_t stat,
                                         uint32_t qtp, float sl2, int kv, Hook hook) {
  constexpr int NC = D / 32, NG = D / 16;  // NG groups of four MFMAs per product
  constexpr int EP = 128 / D;              // elements per MFMA: 1 (D = 128) or 2
  const uint32_t q_row = qt + ad.row, d_row = dt + ad.row, p_tr = qtp + ad.tr, d_tr = dt + ad.tr;
  // A fragment u of the half's 4 NG: Q rows (group 2 c + qb), Q^T of the half before, dO rows, dO^T
  auto frag = [&](auto uc) __attribute__((always_inline)) {
    constexpr int p = uc / NG, f = uc % NG;
    if constexpr (p == 0) {
      return lds_ld8(xor_here<64 * (f / 2)>(q_row) + (f % 2) * 32 * D);
    } else if constexpr (p == 2) {
      return lds_ld8(xor_here<64 * (f % NC)>(d_row) + (f / NC) * 32 * D);
    } else {
      const uint32_t x = xor_here<32 * f>(p == 1 ? p_tr : d_tr);
      return cat8(lds_ld_tr(x), lds_ld_tr(x + 32 * D));
    }
  };
  const uint32_t lstat = stat + ((threadIdx.x & 63) >> 4) * 16;
  floatx4 l4[2], nd4[2];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    l4[qb] = lds_ld4f(lstat + qb * 64);
    nd4[qb] = lds_ld4f(lstat + 256 + qb * 64);
  }
  floatx4 s[8], dp[8];  // block 4 qb + kb: queries 16 qb .. + 15, key block kb
  bf16x8 pb[4];
  // step x of the exponentials: scale and shift (even x), then exp2 and the pack of every second
  // element (odd) of element x / 2
  auto soft = [&](int x) {
    const int e = x / 2, b = e / 4, i = e % 4, kb = b % 4, qb = b / 4;
    if (x % 2 == 0) {
      s[b][i] = fmaf(s[b][i], sl2, -l4[qb][i]);
    } else {
      float y = fast_exp2(s[b][i]);
      if constexpr (kRange) y = (kv >> kb) & 1 ? y : 0.f;
      s[b][i] = y;
      if (i & 1) {
        pb[kb][4 * qb + i - 1] = (__bf16)s[b][i - 1];
        pb[kb][4 * qb + i] = (__bf16)s[b][i];
      }
    }
  };
  auto dsel = [&](int e) {
    const int b = e / 4, i = e % 4, kb = b % 4, qb = b / 4;
    dp[b][i] = s[b][i] * dp[b][i];
    if (i & 1) {
      st.ds[kb][4 * qb + i - 1] = (__bf16)dp[b][i - 1];
      st.ds[kb][4 * qb + i] = (__bf16)dp[b][i];
    }
  };
  bf16x8 fr[4 * NG + kDkvLook];
  bf16x8 kl[NC > kRegChunks ? NC : 1][4];
  static_for<kDkvLook>([&](auto uc) __attribute__((always_inline)) { fr[uc] = frag(uc); });
  static_for<4 * NG>([&](auto uc) __attribute__((always_inline)) {
    constexpr int u = uc, p = u / NG, f = u % NG;
    if constexpr (u + kDkvLook < 4 * NG) fr[u + kDkvLook] = frag(std::integral_constant<int, u + kDkvLook>{});
    // K fragments from LDS, two per group, for the 32 head dims after these
    if constexpr (p == 0 && f / 2 + 1 >= kRegChunks && f / 2 + 1 < NC) {
      constexpr int c = f / 2 + 1, kb = 2 * (f % 2);
      const uint32_t x = xor_here<64 * (c - kRegChunks)>(ad.k);
      kl[c][kb] = lds_ld8(x + kb * 16 * 128);
      kl[c][kb + 1] = lds_ld8(x + (kb + 1) * 16 * 128);
    }
    static_for<4>([&](auto kc) __attribute__((always_inline)) {
      constexpr int kb = kc, x = (4 * f + kb) * EP;
      if constexpr (p == 0) {
        constexpr int c = f / 2, b = 4 * (f % 2) + kb;
        bf16x8 k;
        if constexpr (c < kRegChunks) k = st.kf[kb][c];
        else k = kl[c][kb];
        s[b] = mfma16(fr[u], k, c == 0 ? floatx4{} : s[b]);
      } else if constexpr (p == 1) {
        if constexpr (f == 0) mfma16_agpr(st.dk[kb][f], fr[u], st.ds[kb]);
        else mfma16_agpr_settled(st.dk[kb][f], fr[u], st.ds[kb]);
      } else if constexpr (p == 2) {
        constexpr int c = f % NC, b = 4 * (f / NC) + kb;
        dp[b] = mfma16(fr[u], st.vf[kb][c], c == 0 ? nd4[f / NC] : dp[b]);
      } else {
        if constexpr (f == 0) mfma16_agpr(st.dv[kb][f], fr[u], pb[kb]);
        else mfma16_agpr_settled(st.dv[kb][f], fr[u], pb[kb]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < EP; ++e) {
        if (p == 1) soft(x + e);
        else if (p == 2) soft(32 + x + e);
        else if (p == 3) dsel(x + e);
      }
      if (kb == 1) hook(u);
      __builtin_amdgcn_sched_barrier(0);
    });
  });
}

// Walks the 64-row tiles (the last of a span may be short) of the spans that reach every key of
// the item (kRange: of those that reach only some).
template <bool kRange>
struct QueryCursor {
  const Span* spans;
  int n, si, off, cur_stream, cur_start, cur_len, cur_keys;
  __device__ __forceinline__ void settle() {
    for (; si < n; ++si) {
      const Span s = spans[si];
      cur_keys = __builtin_amdgcn_readfirstlane(s.keys);
      if ((cur_keys != 0) != kRange) continue;
      cur_stream = __builtin_amdgcn_readfirstlane(s.stream);
      cur_start = __builtin_amdgcn_readfirstlane(s.start);
      cur_len = __builtin_amdgcn_readfirstlane(s.len);
      return;
    }
  }
  __device__ __forceinline__ int init(const Span* s, int count) {  // returns the number of tiles
    spans = s;
    n = count;
    int t = 0;
    for (int i = 0; i < count; ++i)
      if ((__builtin_amdgcn_readfirstlane(s[i].keys) != 0) == kRange)
        t += (__builtin_amdgcn_readfirstlane(s[i].len) + kDkvTile - 1) / kDkvTile;
    si = off = 0;
    settle();
    return t;
  }
  __device__ __forceinline__ void advance() {
    off += kDkvTile;
    if (off >= cur_len) {
      ++si;
      off = 0;
      settle();
    }
  }
};

// LDS of a workgroup: the query tiles (Q, dO, LSE and -D per row) and, for d = 128, K's upper dims.
template <int D>
struct DkvLds {
  static constexpr uint32_t kTile = SwzTile<D, kDkvTile>::kElems * 2;
  static constexpr uint32_t kBuf = 2 * kTile + 2 * kDkvTile * 4;
  static constexpr uint32_t kK = D > 64 ? kDkvKeyTile * 128 : 0;
  static constexpr uint32_t kBytes = kDkvBufs * kBuf + kK;
};

// The query tiles of one kind of spans (see QueryCursor), through the pipeline.
template <int D, bool kOneStride, bool kRange>
__device__ __forceinline__ void dkv_spans(const BwdArgs& a, const WorkItem& it, DkvState<D>& st, const DkvAddr& ad,
                                          uint32_t lds0, const uint32_t* qoff, uint32_t doff, int wave, bool active) {
  using L = DkvLds<D>;
  using TL = SwzTile<D, kDkvTile>;
  constexpr int NB = kDkvBufs, kLoads = TL::kInstr / kDkvWaves, NW = kDkvWaves;
  const int lane = threadIdx.x & 63;
  const int h = it.head;
  const float sl2 = a.scale_log2;
  const int64_t dstride = int64_t(a.heads) * D;
  QueryCursor<kRange> ld, cu;
  const Span* sp = a.spans + it.span_off;
  const int T = ld.init(sp, it.span_cnt);
  if (T == 0) return;
  cu.init(sp, it.span_cnt);
  const uint64_t qb0 = uniform_u64(reinterpret_cast<uint64_t>(a.q[0]));
  const uint64_t qb1 = uniform_u64(reinterpret_cast<uint64_t>(a.q[1]));
  const uint64_t db0 = uniform_u64(reinterpret_cast<uint64_t>(a.dout[0]));
  const uint64_t db1 = uniform_u64(reinterpret_cast<uint64_t>(a.dout[1]));
  const uint64_t lb0 = uniform_u64(reinterpret_cast<uint64_t>(wave == 0 ? a.lse2[0] : a.ndelta[0]));
  const uint64_t lb1 = uniform_u64(reinterpret_cast<uint64_t>(wave == 0 ? a.lse2[1] : a.ndelta[1]));
  const int64_t qst0 = a.in_stride[0], qst1 = a.in_stride[1];
  const int hr0 = h * a.rows[0], hr1 = h * a.rows[1];

  // the pending tile load
  uint64_t lq = 0, ldo = 0, lstat = 0, qstep = 0;
  const uint64_t dstep = uint64_t(dstride) * (2 * NW * TL::kRowsPerInstr);
  uint32_t lqoff = 0, lbuf = 0;
  bool lfull = false;
  auto prepare = [&](int b) __attribute__((always_inline)) {  // the next tile -> buffer b
    const int ss = ld.cur_stream;
    const int64_t row0 = ld.cur_start + ld.off, qst = ss ? qst1 : qst0;
    lbuf = lds0 + b * L::kBuf;
    lfull = ld.off + kDkvTile <= ld.cur_len;
    if (lfull) {
      lq = (ss ? qb1 : qb0) + uint64_t(row0 * qst) * 2;
      ldo = (ss ? db1 : db0) + uint64_t(row0 * dstride) * 2;
      lstat = (ss ? lb1 : lb0) + uint64_t(int64_t(ss ? hr1 : hr0) + row0) * 4;
      qstep = uint64_t(qst) * (2 * NW * TL::kRowsPerInstr);
      lqoff = kOneStride || !ss ? qoff[0] : qoff[kOneStride ? 0 : 1];
    } else {
      swz_load_clamped<D, kDkvTile, NW>(lbuf, ss ? qb1 : qb0, qst, h, ld.cur_start, ld.cur_len, ld.off, wave);
      swz_load_clamped<D, kDkvTile, NW>(lbuf + L::kTile, ss ? db1 : db0, dstride, h, ld.cur_start, ld.cur_len, ld.off,
                                        wave);
      if (wave < 2) {  // rows past the span: LSE = +inf (P = 0), -D = 0
        const bool in = ld.off + lane < ld.cur_len;
        const float* src = reinterpret_cast<const float*>(ss ? lb1 : lb0) + (ss ? hr1 : hr0) + ld.cur_start;
        const float x = src[min(ld.off + lane, ld.cur_len - 1)];
        lds_st_f(lbuf + 2 * L::kTile + wave * 256 + lane * 4, in ? x : wave == 0 ? INFINITY : 0.f);
      }
    }
    ld.advance();
  };
  auto load = [&](int j) __attribute__((always_inline)) {  // load j of 2 kLoads + 1 of the pending tile
    if (!lfull) return;
    if (j < kLoads) lds_dma_x4_off(lq + j * qstep, lqoff, lbuf + (wave + j * NW) * 1024);
    else if (j < 2 * kLoads) lds_dma_x4_off(ldo + (j - kLoads) * dstep, doff, lbuf + L::kTile + (wave + (j - kLoads) * NW) * 1024);
    else if (wave < 2) lds_dma_x1_off(lstat, lane * 4, lbuf + 2 * L::kTile + wave * 256);
  };
  __syncthreads();  // every wave is done with the buffers
  prepare(0);
#pragma unroll
  for (int j = 0; j <= 2 * kLoads; ++j) load(j);
  wait_vmem();
  __syncthreads();
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) st.ds[kb] = bf16x8{};  // the half before the first adds 0

  // Tile t sits in buffer t % NB; iteration t loads tile t + 1 into buffer (t + 1) % NB, last read
  // (as the half before tile t - 1's first) in iteration t - 1, before the barrier that ended it.
  uint32_t qtp = lds0;
  int b = 0;
  for (int t = 0; t < T; ++t) {
    const uint32_t qt = lds0 + b * L::kBuf;
    const int n = cu.cur_len - cu.off;
    int kv = 15;
    if constexpr (kRange) {
      const int lo = cu.cur_keys & 0xffff, hi = cu.cur_keys >> 16, key = wave * 64 + (lane & 15);
      kv = 0;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) kv |= (key + 16 * kb >= lo && key + 16 * kb < hi) ? 1 << kb : 0;
    }
    cu.advance();
    b = b + 1 == NB ? 0 : b + 1;
    lfull = false;
    if (t + 1 < T) prepare(b);
    if (active) {
      // the loads are spread over the groups of MFMAs
      constexpr int kEvery = 4 * (D / 16) / kLoads;
      dkv_half<D, kRange>(st, ad, qt, qt + L::kTile, qt + 2 * L::kTile, qtp, sl2, kv,
                          [&](int u) __attribute__((always_inline)) {
                            if (u % kEvery == 0) load(u / kEvery);
                            if (u == 2) load(2 * kLoads);
                          });
      qtp = qt;
    }
    if (active && n > 32) {
      constexpr int kEvery = 4 * (D / 16) / kLoads;
      dkv_half<D, kRange>(st, ad, qt + 64 * D, qt + L::kTile + 64 * D, qt + 2 * L::kTile + 128, qtp, sl2, kv,
                          [&](int u) __attribute__((always_inline)) {
                            if (u % kEvery == 0) load(kLoads + u / kEvery);
                          });
      qtp = qt + 64 * D;
    } else {
#pragma unroll
      for (int j = 0; j <= 2 * kLoads; ++j)
        if (!active || (j >= kLoads && j < 2 * kLoads)) load(j);
    }
    wait_vmem();
    __syncthreads();
  }
  if (active) {  // dK of the last half
#pragma unroll
    for (int f = 0; f < D / 16; ++f) {
      const uint32_t x = (qtp + ad.tr) ^ (32 * f);
      const bf16x8 tf = cat8(lds_ld_tr(x), lds_ld_tr(x + 32 * D));
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) mfma16_agpr(st.dk[kb][f], tf, st.ds[kb]);
    }
  }
}

// One work item; `lds` holds DkvLds<D>::kBytes. kOneStride: gen and ref q share one token stride, so
// one load offset serves both.
template <int D, bool kOneStride>
__device__ __forceinline__ void dkv_item(const BwdArgs& a, const WorkItem& it, const unsigned char* lds) {
  constexpr int NC = D / 32, ND = D / 16;
  using L = DkvLds<D>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, l16 = lane & 15;
  const int h = it.head, s = it.stream;
  const bool active = wave * 64 < it.len;
  const int64_t dstride = int64_t(a.heads) * D;
  const uint32_t lds0 = lds_addr(lds), kl0 = lds0 + kDkvBufs * L::kBuf;

  // the item's keys: V and K fragments into VGPRs, K's upper head dims into LDS as a 64-dim tile
  // (rows clamped at the tile end)
  if constexpr (D > 64)
    swz_load_clamped<64, kDkvKeyTile, kDkvWaves>(kl0, reinterpret_cast<uint64_t>(a.k[s] + h * D + 64), a.in_stride[s], 0,
                                                 it.start, it.len, 0, wave);
  DkvState<D> st;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    const int r = wave * 64 + 16 * kb + l16;
    const int64_t off = int64_t(it.start + min(r, it.len - 1)) * a.in_stride[s] + h * D + g * 8;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const bf16x8 y = ld8(a.v[s] + off + c * 32);
      st.vf[kb][c] = (r < it.len) ? y : bf16x8{};
      if (c < kRegChunks) st.kf[kb][c] = ld8(a.k[s] + off + c * 32);
    }
#pragma unroll
    for (int db = 0; db < ND; ++db) st.dk[kb][db] = st.dv[kb][db] = floatx4{};
  }
  // land them here: left to their first use, which is inside the loop, the compiler would wait
  // there, each time round, for every direct load in flight too
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
#pragma unroll
    for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(st.vf[kb][c]));
#pragma unroll
    for (int c = 0; c < kRegChunks; ++c) asm volatile("" : "+v"(st.kf[kb][c]));
  }
  const DkvAddr ad{swz_row_addr<D>(), swz_tr_addr<D>(), kl0 + uint32_t(wave) * 64 * 128 + swz_row_addr<64>()};
  uint32_t qoff[kOneStride ? 1 : 2];
#pragma unroll
  for (int ss = 0; ss < (kOneStride ? 1 : 2); ++ss) qoff[ss] = swz_load_off<D>(a.in_stride[ss], h, wave);
  const uint32_t doff = swz_load_off<D>(dstride, h, wave);

  dkv_spans<D, kOneStride, false>(a, it, st, ad, lds0, qoff, doff, wave, active);
  dkv_spans<D, kOneStride, true>(a, it, st, ad, lds0, qoff, doff, wave, active);
  mfma_drain();
  // the sums are read only behind the wait (volatile statements keep their order)
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int db = 0; db < ND; ++db) asm volatile("" : "+a"(st.dk[kb][db]), "+a"(st.dv[kb][db]));

  if (!active) return;
  float* part = it.slot ? a.part_kv + int64_t(it.slot - 1) * 2 * kDkvKeyTile * D : nullptr;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    const int r = wave * 64 + 16 * kb + l16;
    if (r >= it.len) continue;
    if (part) {  // a piece of a split item
      float* p = part + r * D + 4 * g;
#pragma unroll
      for (int db = 0; db < ND; ++db) {
        *reinterpret_cast<floatx4*>(p + db * 16) = st.dk[kb][db];
        *reinterpret_cast<floatx4*>(p + kDkvKeyTile * D + db * 16) = st.dv[kb][db];
      }
      continue;
    }
    __bf16* kout = a.dk[s] + int64_t(it.start + r) * dstride + h * D;
    __bf16* vout = a.dv[s] + int64_t(it.start + r) * dstride + h * D;
#pragma unroll
    for (int db = 0; db < ND; ++db) {
      bf16x4 wk, wv;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        wk[e] = (__bf16)(st.dk[kb][db][e] * a.scale);
        wv[e] = (__bf16)(st.dv[kb][db][e]);
      }
      *reinterpret_cast<bf16x4*>(kout + db * 16 + 4 * g) = wk;
      *reinterpret_cast<bf16x4*>(vout + db * 16 + 4 * g) = wv;
    }
  }
}

}  // namespace sra
