// dQ work items of the SRA backward on gfx950 (the gradient is described in sra_bwd.hip).
//
// Query-major, like the forward: a work item is a tile of 256 query rows of one stream and
// head; its four waves (one per SIMD) own 64 rows each, as four 16-row MFMA blocks, and keep
// those rows' Q and dO as B fragments in registers and their dQ sums in AGPRs. The key rows the
// queries see (the spans of the query-major schedule) stream through LDS in 64-row tiles, taken
// as two 32-key halves, and S and P are recomputed from the forward's log-sum-exp:
//     S^T = K Q^T, dP^T = V dO^T, dS^T = P^T (dP^T - D), dQ^T += K^T dS^T.
// Each K and V fragment read from LDS feeds all four row blocks of a wave. A half's dQ product
// runs behind the next half's S product, so that every product has vector work to hide: dS of
// the half before during S, the exponentials during dQ and dP. Built with MFMAs in VGPR form;
// the dQ products are AGPR-accumulating MFMAs (mfma16_agpr). Bound by the clock that the board's power
// allows (720p: 1.99 of 2.4 GHz) and by issue: the MFMA pipes are busy 63 % of the cycles, with 1.4 vector
// instructions per MFMA; waves wait for an issue slot in 25 % of their cycles, for data in 16 %.
// 480p, 5 heads 5.83 ms with 32x32x16 MFMAs in 32-key tiles, 5.00 ms so.
#pragma once
#include "sra_kernels.h"
#include "sra_tiles.h"

namespace sra {

constexpr int kDqWaves = kDqQueryTile / 64;  // one wave per SIMD, 64 query rows each
constexpr int kDqTile = 64;                  // keys per LDS tile
constexpr int kDqBufs = 4;
constexpr int kDqLook = 2;   // LDS fragments are read this many groups of four MFMAs ahead

template <int D>
struct DqState {
  bf16x8 qf[4][D / 32];   // Q^T B fragments of the four 16-row blocks (lane = query)
  bf16x8 df[4][D / 32];   // dO^T B fragments
  floatx4 dq[4][D / 16];  // dQ^T accumulators (lane = query), 16 head dims each
  floatx4 nd[4];          // -rowsum(dO * O) of the row, four times: dP's starting value
  float lse2[4];          // the rows' log-sum-exp (log2 units)
  // of the half before: P and dP - D of its keys 16..31 (row blocks qb), and the dS fragments,
  // whose elements 0..3 (keys 0..15) are done
  floatx4 p1[4], dp1[4];
  bf16x8 ds[4];
  bf16x8 ah[kDqLook];     // the next half's first K fragments
};

// LDS byte addresses of a wave's fragments: row fragments of c = 0 and transpose reads of db = 0
// (the others by XOR), for a tile at LDS address 0.
struct DqAddr {
  uint32_t row, tr;
};

// dS of element e (of 16) of 16 keys, from P and dP - D, packed in pairs into elements
// 4 kb .. + 3 of the B fragments of the dQ product.
__device__ __forceinline__ void dq_ds(floatx4 p[4], floatx4 dp[4], bf16x8 ds[4], int kb, int e) {
  const int qb = e / 4, i = e % 4;
  dp[qb][i] = p[qb][i] * dp[qb][i];
  if (i & 1) {
    ds[qb][4 * kb + i - 1] = (__bf16)dp[qb][i - 1];
    ds[qb][4 * kb + i] = (__bf16)dp[qb][i];
  }
}

// One 32-key half for the wave's 64 query rows: S of this half, dQ of the half before, dP of this
// half. kt, vt: LDS addresses of this half's K and V rows; ktp, ktn: of the K
// rows of the halves before and after.
// Each MFMA is followed by its share of the vector work (a 16x16x32 MFMA hides about 8 cycles of
// it) and a scheduling barrier: dS of the half before's keys 16..31 under S of keys 0..15, the
// exponentials from there to dP of keys 0..15, dS of keys 0..15 under dP of keys 16..31. LDS
// fragments are read kDqLook groups of four MFMAs ahead, across halves too.
// hook(u) runs behind MFMA group u = 0 .. 3 D / 16 - 1 (the direct loads of the next tile).
template <int D, class Hook>
__device__ __forceinline__ void dq_half(DqState<D>& st, const DqAddr& ad, uint32_t kt, uint32_t vt, uint32_t ktp,
                                        uint32_t ktn, float sl2, Hook hook) {
  constexpr int NC = D / 32, NG = D / 16;  // NG groups of four MFMAs per product
  constexpr int EP = 128 / D;              // elements per MFMA: 1 (D = 128) or 2
  const uint32_t k_row = kt + ad.row, v_row = vt + ad.row, n_row = ktn + ad.row, p_tr = ktp + ad.tr;
  // fragment u of the half's 3 NG (K rows, K^T of the half before, V rows) and the next half's first
  auto frag = [&](auto uc) __attribute__((always_inline)) {
    constexpr int p = uc / NG, f = uc % NG;
    if constexpr (p == 1) {
      const uint32_t x = xor_here<32 * f>(p_tr);
      return cat8(lds_ld_tr(x), lds_ld_tr(x + 32 * D));
    } else {
      return lds_ld8(xor_here<64 * (f % NC)>(p == 0 ? k_row : p == 2 ? v_row : n_row) + (f / NC) * 32 * D);
    }
  };
  bf16x8 fr[3 * NG + kDqLook];
#pragma unroll
  for (int i = 0; i < kDqLook; ++i) fr[i] = st.ah[i];
  // step x of the exponentials: scale and shift (even x), then exp2 (odd) of element x / 2
  floatx4 s[8], dp[8];
  auto soft = [&](int x) {
    const int e = x / 2, b = e / 4, i = e % 4;
    if (x % 2 == 0) s[b][i] = fmaf(s[b][i], sl2, -st.lse2[b % 4]);
    else s[b][i] = fast_exp2(s[b][i]);
  };
  static_for<3 * NG>([&](auto uc) __attribute__((always_inline)) {
    constexpr int u = uc, p = u / NG, f = u % NG;
    fr[u + kDqLook] = frag(std::integral_constant<int, u + kDqLook>{});
    static_for<4>([&](auto qc) __attribute__((always_inline)) {
      constexpr int qb = qc, b = 4 * (f / NC) + qb, c = f % NC, x = (4 * f + qb) * EP;
      if constexpr (p == 0) s[b] = mfma16(fr[u], st.qf[qb][c], c == 0 ? floatx4{} : s[b]);  // S^T = K Q^T
      else if constexpr (p == 1 && f == 0) mfma16_agpr(st.dq[qb][f], fr[u], st.ds[qb]);
      else if constexpr (p == 1) mfma16_agpr_settled(st.dq[qb][f], fr[u], st.ds[qb]);               // dQ^T += K^T dS^T
      else dp[b] = mfma16(fr[u], st.df[qb][c], c == 0 ? st.nd[qb] : dp[b]);                 // dP^T - D
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < EP; ++e) {
        const int y = x + e;  // of 32 in each product
        if (p == 0) {
          if (y < 16) dq_ds(st.p1, st.dp1, st.ds, 1, y);
          else soft(y - 16);
        } else if (p == 1) {
          soft(16 + y);
        } else {
          if (y < 16) soft(48 + y);
          else dq_ds(s, dp, st.ds, 0, y - 16);
        }
      }
      if (qb == 1) hook(u);
      __builtin_amdgcn_sched_barrier(0);
    });
  });
#pragma unroll
  for (int i = 0; i < kDqLook; ++i) st.ah[i] = fr[3 * NG + i];
#pragma unroll
  for (int qb = 0; qb < 4; ++qb) {
    st.p1[qb] = s[4 + qb];
    st.dp1[qb] = dp[4 + qb];
  }
}

// dQ^T += K^T dS^T of the half before (its dS still to be finished for keys 16..31).
template <int D>
__device__ __forceinline__ void dq_flush(DqState<D>& st, const DqAddr& ad, uint32_t ktp) {
#pragma unroll
  for (int e = 0; e < 16; ++e) dq_ds(st.p1, st.dp1, st.ds, 1, e);
#pragma unroll
  for (int db = 0; db < D / 16; ++db) {
    const uint32_t x = (ktp + ad.tr) ^ (32 * db);
    const bf16x8 tf = cat8(lds_ld_tr(x), lds_ld_tr(x + 32 * D));
#pragma unroll
    for (int qb = 0; qb < 4; ++qb) mfma16_agpr(st.dq[qb][db], tf, st.ds[qb]);
  }
}

// One 32-key half, plain, for the ragged ends of spans: keys >= nvalid are outside the span.
template <int D>
__device__ __forceinline__ void dq_masked(DqState<D>& st, const DqAddr& ad, uint32_t kt, uint32_t vt, int nvalid,
                                          float sl2) {
  constexpr int NC = D / 32;
  const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    floatx4 s[4], dp[4];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const bf16x8 ka = lds_ld8(((kt + ad.row) ^ (64 * c)) + kb * 32 * D);
      const bf16x8 va = lds_ld8(((vt + ad.row) ^ (64 * c)) + kb * 32 * D);
#pragma unroll
      for (int qb = 0; qb < 4; ++qb) {
        s[qb] = mfma16(ka, st.qf[qb][c], c == 0 ? floatx4{} : s[qb]);
        dp[qb] = mfma16(va, st.df[qb][c], c == 0 ? st.nd[qb] : dp[qb]);
      }
    }
#pragma unroll
    for (int qb = 0; qb < 4; ++qb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = fast_exp2(fmaf(s[qb][i], sl2, -st.lse2[qb]));
        s[qb][i] = (16 * kb + 4 * g + i) < nvalid ? p : 0.f;
      }
    if (kb == 0) {
#pragma unroll
      for (int e = 0; e < 16; ++e) dq_ds(s, dp, st.ds, 0, e);
    } else {
#pragma unroll
      for (int qb = 0; qb < 4; ++qb) {
        st.p1[qb] = s[qb];
        st.dp1[qb] = dp[qb];
      }
    }
  }
  dq_flush<D>(st, ad, kt);
}

template <int D>
constexpr uint32_t kDqLdsBytes = kDqBufs * 2 * SwzTile<D, kDqTile>::kElems * 2;

// One work item; `lds` holds kDqLdsBytes<D>. kOneStride: the streams share one token stride, so one
// load offset serves both.
template <int D, bool kOneStride>
__device__ __forceinline__ void dq_item(const BwdArgs& a, const WorkItem& it, const unsigned char* lds) {
  constexpr int NC = D / 32, ND = D / 16, BK = kDqTile, NB = kDqBufs;
  using TL = SwzTile<D, BK>;
  constexpr uint32_t kTileBytes = TL::kElems * 2;
  constexpr int kLoads = TL::kInstr / kDqWaves;  // of K, and of V, per wave and tile

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, l16 = lane & 15;
  const int h = it.head, s = it.stream & 1;
  const bool active = wave * 64 < it.len;
  const float sl2 = a.scale_log2;
  const int64_t dstride = int64_t(a.heads) * D;

  const Span* sp = a.spans + it.span_off;
  int T = 0;  // full tiles over all spans
  for (int i = 0; i < it.span_cnt; ++i) T += __builtin_amdgcn_readfirstlane(sp[i].len) / BK;
  FullTileCursor<BK> ld;  // next full tile to load
  ld.init(sp, it.span_cnt);
  const uint64_t kb0 = uniform_u64(reinterpret_cast<uint64_t>(a.k[0]));
  const uint64_t kb1 = uniform_u64(reinterpret_cast<uint64_t>(a.k[1]));
  const uint64_t vb0 = uniform_u64(reinterpret_cast<uint64_t>(a.v[0]));
  const uint64_t vb1 = uniform_u64(reinterpret_cast<uint64_t>(a.v[1]));
  const int64_t st0 = a.in_stride[0], st1 = a.in_stride[1];
  uint32_t voff[kOneStride ? 1 : 2];
#pragma unroll
  for (int ss = 0; ss < (kOneStride ? 1 : 2); ++ss) voff[ss] = swz_load_off<D>(a.in_stride[ss], h, wave);
  const uint32_t lds0 = lds_addr(lds);

  // the pending tile load: bases and LDS address of this wave's instructions
  uint64_t lk = 0, lv = 0, lstep = 0;
  uint32_t lvoff = 0, lla = 0;
  auto prepare = [&](int b) __attribute__((always_inline)) {  // the next full tile -> buffer b
    const int ss = ld.cur_stream;
    const int64_t st = ss ? st1 : st0;
    lla = lds0 + b * 2 * kTileBytes + wave * 1024;
    const uint64_t row0 = uint64_t(int64_t(ld.cur_start + ld.off) * st) * 2;
    lk = (ss ? kb1 : kb0) + row0;
    lv = (ss ? vb1 : vb0) + row0;
    lstep = uint64_t(st) * (2 * kDqWaves * TL::kRowsPerInstr);
    lvoff = kOneStride || !ss ? voff[0] : voff[kOneStride ? 0 : 1];
    ld.advance();
  };
  auto load = [&](int j) __attribute__((always_inline)) {  // load j of 2 kLoads of the pending tile
    if (j < kLoads) lds_dma_x4_off(lk + j * lstep, lvoff, lla + j * kDqWaves * 1024);
    else lds_dma_x4_off(lv + (j - kLoads) * lstep, lvoff, lla + kTileBytes + (j - kLoads) * kDqWaves * 1024);
  };
  for (int b = 0; b < 2 && b < T; ++b) {
    prepare(b);
#pragma unroll
    for (int j = 0; j < 2 * kLoads; ++j) load(j);
  }

  DqState<D> st;
#pragma unroll
  for (int qb = 0; qb < 4; ++qb) {
    const int r = wave * 64 + 16 * qb + l16;
    const int rr = it.start + min(r, it.len - 1);
    const __bf16* qp = a.q[s] + int64_t(rr) * a.in_stride[s] + h * D + g * 8;
    const __bf16* dp = a.dout[s] + int64_t(rr) * dstride + h * D + g * 8;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const bf16x8 x = ld8(qp + c * 32);
      const bf16x8 y = ld8(dp + c * 32);
      st.qf[qb][c] = (r < it.len) ? x : bf16x8{};
      st.df[qb][c] = (r < it.len) ? y : bf16x8{};
    }
#pragma unroll
    for (int db = 0; db < ND; ++db) st.dq[qb][db] = floatx4{};
    st.lse2[qb] = a.lse2[s][int64_t(h) * a.rows[s] + rr];
    const float n = a.ndelta[s][int64_t(h) * a.rows[s] + rr];
    st.nd[qb] = floatx4{n, n, n, n};
  }
#pragma unroll
  for (int qb = 0; qb < 4; ++qb) {  // the half before the first adds 0
    st.p1[qb] = st.dp1[qb] = floatx4{};
    st.ds[qb] = bf16x8{};
  }
  // land the rows' loads here: left to their first use, which is inside the loop, the compiler
  // would wait there, each time round, for every direct load in flight too
#pragma unroll
  for (int qb = 0; qb < 4; ++qb) {
#pragma unroll
    for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(st.qf[qb][c]), "+v"(st.df[qb][c]));
    asm volatile("" : "+v"(st.lse2[qb]), "+v"(st.nd[qb]));
  }
  const DqAddr ad{swz_row_addr<D>(), swz_tr_addr<D>()};
  wait_vmem();
  __syncthreads();

  // Tile t sits in buffer t % NB; iteration t loads tile t + 2 into buffer (t + 2) % NB, last read
  // (as the half before tile t - 1's first) in iteration t - 1, before the barrier that ended it.
  // Its end waits for its loads, so tile t + 1 has landed before iteration t begins and its first
  // fragments can be read during it. The last two iterations load the last tile again, into
  // buffers that nothing reads by then.
  if (T > 0) {
    uint32_t ktp = lds0;
    int b = 0, bl = T > 1 ? 2 : 1;
#pragma unroll
    for (int i = 0; i < kDqLook; ++i) st.ah[i] = lds_ld8(((lds0 + ad.row) ^ (64 * (i % NC))) + (i / NC) * 32 * D);
    for (int t = 0; t < T; ++t) {
      const uint32_t kt = lds0 + b * 2 * kTileBytes, vt = kt + kTileBytes;
      b = (b + 1) % NB;
      const uint32_t ktn = lds0 + b * 2 * kTileBytes;
      if (t + 2 < T) prepare(bl);
      else lla = lds0 + bl * 2 * kTileBytes + wave * 1024;
      bl = (bl + 1) % NB;
      if (active) {
        // the loads are spread over the first half's groups of MFMAs, the second half covers them
        constexpr int kEvery = 3 * (D / 16) / (2 * kLoads);
        dq_half<D>(st, ad, kt, vt, ktp, kt + 64 * D, sl2, [&](int u) __attribute__((always_inline)) {
          if (u % kEvery == 0 && u / kEvery < 2 * kLoads) load(u / kEvery);
        });
        dq_half<D>(st, ad, kt + 64 * D, vt + 64 * D, kt, ktn, sl2, [](int) {});
        ktp = kt + 64 * D;
      } else {
#pragma unroll
        for (int j = 0; j < 2 * kLoads; ++j) load(j);
      }
      wait_vmem();
      block_barrier();
    }
    if (active) dq_flush<D>(st, ad, ktp);
  }
  // ragged ends of the spans
  for (int i = 0; i < it.span_cnt; ++i) {
    const Span x = sp[i];
    const int len = __builtin_amdgcn_readfirstlane(x.len), rem = len % BK;
    if (rem == 0) continue;
    __syncthreads();  // every wave is done with the buffers
    const int ss = __builtin_amdgcn_readfirstlane(x.stream), start = __builtin_amdgcn_readfirstlane(x.start);
    swz_load_clamped<D, BK, kDqWaves>(lds0, ss ? kb1 : kb0, ss ? st1 : st0, h, start, len, len - rem, wave);
    swz_load_clamped<D, BK, kDqWaves>(lds0 + kTileBytes, ss ? vb1 : vb0, ss ? st1 : st0, h, start, len, len - rem, wave);
    wait_vmem();
    __syncthreads();
    if (active)
      for (int o = 0; o < rem; o += 32) dq_masked<D>(st, ad, lds0 + o * 2 * D, lds0 + kTileBytes + o * 2 * D, rem - o, sl2);
  }
  mfma_drain();
  // the sums are read only behind the wait (volatile statements keep their order)
#pragma unroll
  for (int qb = 0; qb < 4; ++qb)
#pragma unroll
    for (int db = 0; db < ND; ++db) asm volatile("" : "+a"(st.dq[qb][db]));

  if (!active) return;
  float* part = it.slot ? a.part_q + int64_t(it.slot - 1) * kDqQueryTile * D : nullptr;
#pragma unroll
  for (int qb = 0; qb < 4; ++qb) {
    const int r = wave * 64 + 16 * qb + l16;
    if (r >= it.len) continue;
    if (part) {  // a piece of a split item
#pragma unroll
      for (int db = 0; db < ND; ++db) *reinterpret_cast<floatx4*>(part + r * D + db * 16 + 4 * g) = st.dq[qb][db];
      continue;
    }
    __bf16* orow = a.dq[s] + int64_t(it.start + r) * dstride + h * D;
#pragma unroll
    for (int db = 0; db < ND; ++db) {
      bf16x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = (__bf16)(st.dq[qb][db][e] * a.scale);
      *reinterpret_cast<bf16x4*>(orow + db * 16 + 4 * g) = w;
    }
  }
}

}  // namespace sra
