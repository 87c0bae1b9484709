// Forward pass of Sparse Reference Attention on gfx950.
//
// One workgroup (8 wave64s, two per SIMD) takes one work item: a tile of up to 128 NQ (256, 384 or
// 512) query rows of one stream and head, plus the list of key spans those rows see (Avatar V §1,
// §2.1, §4.3: gen rows see the gen keys and the valid ref frames of their sample; ref rows
// see the valid frames of their own group). Every wave owns 16 NQ query rows, as NQ MFMA column
// blocks, and keeps Q^T and O^T in VGPRs; keys stream through LDS in 64-row tiles (direct
// global->LDS loads, three buffers each for K and V):
//
//   S^T (keys x queries) = K Q^T          bf16 MFMA 16x16x32, K row fragments from LDS
//   online softmax over keys in base 2, lanes = queries (row sums are lane-local plus two
//   permlane swaps)
//   O^T (d x queries) += V^T P^T          V^T fragments via the LDS transpose read
//
// 16x16x32 MFMAs: at the board's power limit they sustain 2,050 TFLOP/s from registers on
// random data, 32x32x16 ones 1,840 (one wave per SIMD) or 1,350 (two). Launches that end before that
// limit sets in run on 32x32x16 ones (sra_fwd32.hip).
//
// Bound by the clock that the board's power allows (720p: 1.94 of 2.4 GHz) and by issue: the MFMA pipes
// are busy 65 % of the cycles, with 1.9 vector instructions per MFMA; waves wait for an issue slot in
// 31 % of their cycles, for data or a barrier in 29 %, for LDS in 2 %.
//
// What one 16-row block costs in LDS reads falls with the rows per wave: 32 rows (d = 128, 256-row
// items) feed two MFMAs per fragment, 48 (d = 128) three, 64 (d = 64) four. 480p layer, 40 heads:
// 26.2 ms with 32x32x16 MFMAs, 25.5 with these, 23.8 (1,340 TFLOP/s) with 48 rows.
//
// The key loop is software-pipelined in 32-key halves and each wave's instruction stream is
// laid out by hand: one block issues the P V product of the previous half and the S^T product
// of the next half, slot by slot, each MFMA followed by its share of the softmax of the current
// half; LDS fragments are read one slot pair ahead, across blocks too. A wave's MFMAs then run
// while the same wave issues its softmax arithmetic, instead of the two alternating in phases.
//
// The running max m is not tracked per half. P is computed against the current m, and its
// partial row sum doubles as the overflow check: if some lane's 8 values of a row sum to more
// than kBigSum (some P > kBigSum, or an inf from m = -inf at the start), the wave takes the rare
// slow path: recompute that half's S, set m to the true running max, rescale O and l,
// recompute P. So m always lies within log2(kBigSum) of the true row max.
//
// Full 64-key tiles of all spans run through the pipeline first; the ragged tail of each
// span runs afterwards in a masked, unpipelined step (the accumulation is order-independent).
#include <type_traits>

#include "sra_kernels.h"
#include "sra_tiles.h"

namespace sra {

namespace {
constexpr float kLn2 = 0.69314718055994530942f;
constexpr float kBigSum = 65536.0f;  // a lane's half-step sum of P above this forces a rescale
constexpr int kLook = 1;             // LDS fragments are read this many slot pairs ahead
constexpr int kWaves = 8;
template <int D> using KTile = PaddedTile<D, kFwdKeyStep, kPadRS<D>>;  // row-fragment reads
template <int D> using VTile = PaddedTile<D, kFwdKeyStep, kPadRS<D>>;  // transpose reads
}  // namespace

template <int D, int NQ>
struct FwdState {
  bf16x8 qf[NQ][D / 32];  // Q^T MFMA B fragments of the 16-row blocks: lane = query, 8 head dims
  floatx4 o[NQ][D / 16];  // O^T accumulators, 16 head dims each
  float m[NQ];            // running max (log2 units)
  float l[NQ];            // per-lane partial row sum (fp32)
};

// Scores of a 32-key half for the wave's 16 NQ query rows: b[NQ * kb + qb] holds keys 16 kb .. + 15
// of row block qb. Element e of the flat order is register e % 4 of block e / 4.
template <int NQ>
struct HalfS {
  floatx4 b[2 * NQ];
};

// P of one 32-key half as the B fragments of the P V product, one per row block: elements 0..3
// are keys 4 g + i and elements 4..7 keys 16 + 4 g + i (g = lane / 16), the MFMA output's order.
template <int NQ>
struct HalfP {
  bf16x8 p[NQ];
};

// The first kLook K and V fragments of the next pipelined block, read during the last slots of
// the block before it (their tiles have landed by then, also across the barrier between tiles).
struct Ahead {
  bf16x8 k[kLook], v[kLook];
};

// K row fragment i of the 32 keys at kt (A operand of S^T = K Q^T): keys 16 kb .. + 15 and head
// dims 32 c .. + 31, i = (D / 32) kb + c.
template <int D>
__device__ __forceinline__ bf16x8 k_frag(const __bf16* kt, int i) {
  const int lane = threadIdx.x & 63, kb = i / (D / 32), c = i % (D / 32);
  return *reinterpret_cast<const bf16x8*>(kt + ((lane & 15) + 16 * kb) * kPadRS<D> + c * 32 + (lane >> 4) * 8);
}

// V^T fragment db of the 32 keys at vt (A operand of O^T += V^T P^T): head dims 16 db .. + 15.
// The transpose read gives lane (head dim) the 8 keys whose P values the B fragment holds.
template <int D>
__device__ __forceinline__ bf16x8 v_frag(const __bf16* vt, int db) {
  const int lane = threadIdx.x & 63;
  const int r0 = 4 * (lane >> 4) + ((lane & 15) >> 2), col = db * 16 + 4 * (lane & 3);
  return cat8(lds_read_tr(vt + r0 * kPadRS<D> + col), lds_read_tr(vt + (r0 + 16) * kPadRS<D> + col));
}

// S^T of 32 keys, plain (used outside the pipeline).
template <int D, int NQ>
__device__ __forceinline__ HalfS<NQ> scores32(const FwdState<D, NQ>& st, const __bf16* kt) {
  HalfS<NQ> s;
#pragma unroll
  for (int j = 0; j < 2 * NQ; ++j) s.b[j] = floatx4{};
#pragma unroll
  for (int i = 0; i < D / 16; ++i) {
    const int kb = i / (D / 32), c = i % (D / 32);
    const bf16x8 k = k_frag<D>(kt, i);
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) s.b[NQ * kb + qb] = mfma16(k, st.qf[qb][c], s.b[NQ * kb + qb]);
  }
  return s;
}

template <int NQ>
__device__ __forceinline__ HalfP<NQ> pack_half(const HalfS<NQ>& s) {
  HalfP<NQ> h;
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h.p[qb][i] = (__bf16)s.b[qb][i];
      h.p[qb][4 + i] = (__bf16)s.b[NQ + qb][i];
    }
  return h;
}

// Rare path: s holds S^T of a half (recomputed); move m to the true running max, rescale O
// and l, and leave P of the half in s and the lane's partial sums in sum.
template <int D, int NQ>
__device__ __forceinline__ void rescale_half(FwdState<D, NQ>& st, HalfS<NQ>& s, float sl2, float sum[NQ]) {
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    floatx4& a = s.b[qb];
    floatx4& b = s.b[NQ + qb];
    const float mx = quad_max(max2f(max3f(a[0], a[1], max2f(a[2], a[3])), max3f(b[0], b[1], max2f(b[2], b[3])))) * sl2;
    if (mx > st.m[qb]) {
      const float alpha = fast_exp2(st.m[qb] - mx);  // 0 when m was -inf
      st.m[qb] = mx;
      st.l[qb] *= alpha;
#pragma unroll
      for (int db = 0; db < D / 16; ++db) st.o[qb][db] *= alpha;
    }
    // A row whose scores so far are all -inf (keys masked by an infinite head dim) keeps P = 0, wherever
    // its work item or piece begins.
    const float nm = st.m[qb] == -INFINITY ? 0.f : -st.m[qb];
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = fast_exp2(fmaf(a[i], sl2, nm));
      b[i] = fast_exp2(fmaf(b[i], sl2, nm));
      acc += a[i] + b[i];
    }
    sum[qb] = acc;
  }
}

// The softmax work issued behind MFMA U of a block's 16 NQ (two per element of the half),
// software-pipelined so that instructions issued together never depend on each other: behind an
// even MFMA the exp2 of the element one ahead, behind an odd one the scale-and-shift FMA of the
// element two ahead and the row-sum add (with the bf16 pack of every second one) of element U / 2.
template <int E, int NQ>
__device__ __forceinline__ void soft_fma(HalfS<NQ>& s, const float* nm, float sl2) {
  if constexpr (E < 8 * NQ) s.b[E / 4][E % 4] = fmaf(s.b[E / 4][E % 4], sl2, nm[(E / 4) % NQ]);
}
template <int E, int NQ>
__device__ __forceinline__ void soft_exp(HalfS<NQ>& s) {
  if constexpr (E < 8 * NQ) s.b[E / 4][E % 4] = fast_exp2(s.b[E / 4][E % 4]);
}
template <int U, int NQ>
__device__ __forceinline__ void soft_step(HalfS<NQ>& s, const float* nm, float sl2, float* acc, HalfP<NQ>& out) {
  constexpr int e = U / 2, blk = e / 4, qb = blk % NQ, kb = blk / NQ, i = e % 4;
  if constexpr (U % 2 == 0) {
    soft_exp<e + 1>(s);
  } else {
    soft_fma<e + 2>(s, nm, sl2);
    acc[qb] += s.b[blk][i];
    if constexpr (i & 1) {
      const bf16x2 pr = {(__bf16)s.b[blk][i - 1], (__bf16)s.b[blk][i]};
      out.p[qb][4 * kb + i - 1] = pr[0];
      out.p[qb][4 * kb + i] = pr[1];
    }
  }
}

// MFMA U of a pipelined block (recursion over U): slots of NQ MFMAs sharing one LDS fragment
// alternate S^T of K fragment U / 2 NQ of the next half and P V of V fragment U / 2 NQ of a
// finished half. Each MFMA is followed by its softmax step (a 16x16x32 MFMA of 16 cycles hides
// about 8 cycles of vector work). Fragments LOOK slot pairs ahead are read from LDS. Scheduling
// barriers keep the order.
template <int U, int D, int NQ, int LOOK>
__device__ __forceinline__ void pipe_slots(FwdState<D, NQ>& st, HalfS<NQ>& s_cur, HalfS<NQ>& sn, bf16x8* kf, bf16x8* vf,
                                           const __bf16* kq, const __bf16* vp, const __bf16* kn, const __bf16* vn,
                                           const HalfP<NQ>& pv, const float* nm, float sl2, float* acc,
                                           HalfP<NQ>& out) {
  constexpr int NC = D / 16;
  if constexpr (U < 2 * NC * NQ) {
    constexpr int I = U / (2 * NQ), qb = U % NQ;
    if constexpr (U % (2 * NQ) < NQ) {
      constexpr int kb = I / (D / 32), c = I % (D / 32);
      if constexpr (qb == 0) kf[I + LOOK] = I + LOOK < NC ? k_frag<D>(kq, I + LOOK) : k_frag<D>(kn, I + LOOK - NC);
      sn.b[NQ * kb + qb] = mfma16(kf[I], st.qf[qb][c], c == 0 ? floatx4{} : sn.b[NQ * kb + qb]);
    } else {
      if constexpr (qb == 0) vf[I + LOOK] = I + LOOK < NC ? v_frag<D>(vp, I + LOOK) : v_frag<D>(vn, I + LOOK - NC);
      st.o[qb][I] = mfma16(vf[I], pv.p[qb], st.o[qb][I]);
    }
    __builtin_amdgcn_sched_barrier(0);
    // D = 64 has one MFMA per element: both of an element's steps follow it
    if constexpr (D == 128) {
      soft_step<U>(s_cur, nm, sl2, acc, out);
    } else {
      soft_step<2 * U>(s_cur, nm, sl2, acc, out);
      soft_step<2 * U + 1>(s_cur, nm, sl2, acc, out);
    }
    __builtin_amdgcn_sched_barrier(0);
    pipe_slots<U + 1, D, NQ, LOOK>(st, s_cur, sn, kf, vf, kq, vp, kn, vn, pv, nm, sl2, acc, out);
  }
}

// One pipelined block. MFMA slots alternate S^T = K Q^T of the next half (K rows at kq, into
// s_next) and O^T += V^T P^T of a finished half (V rows at vp, P in pv); after each group of
// MFMAs one slice of the softmax of the current half (s_cur, whose K rows are at kc) is issued.
// Returns P of the current half. Slot order is fixed with scheduling barriers.
template <int D, int NQ>
__device__ __forceinline__ HalfP<NQ> pipe_block(FwdState<D, NQ>& st, HalfS<NQ>& s_cur, const __bf16* kc,
                                                HalfS<NQ>& s_next, const __bf16* kq, const __bf16* vp,
                                                const __bf16* kn, const __bf16* vn, Ahead& ah, const HalfP<NQ>& pv,
                                                float sl2) {
  constexpr int NC = D / 16;  // K fragments of a half (2 x D/32), V fragments of a half (D/16)
  float nm[NQ], acc[NQ];
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    nm[qb] = -st.m[qb];
    acc[qb] = 0.f;
  }
  HalfP<NQ> out;
  bf16x8 kf[NC + kLook], vf[NC + kLook];
#pragma unroll
  for (int i = 0; i < kLook; ++i) {
    kf[i] = ah.k[i];
    vf[i] = ah.v[i];
  }
  HalfS<NQ> sn;
  // prologue of the softmax pipeline: FMA of elements 0 and 1, exp2 of element 0
  soft_fma<0>(s_cur, nm, sl2);
  soft_fma<1>(s_cur, nm, sl2);
  soft_exp<0>(s_cur);
  pipe_slots<0, D, NQ, kLook>(st, s_cur, sn, kf, vf, kq, vp, kn, vn, pv, nm, sl2, acc, out);
  s_next = sn;
#pragma unroll
  for (int i = 0; i < kLook; ++i) {
    ah.k[i] = kf[NC + i];
    ah.v[i] = vf[NC + i];
  }
  // keep the bf16 packs in the slots above (not sunk past the rare-path branch)
  bool ok = true;
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    asm volatile("" : "+v"(out.p[qb]));
    ok = ok && acc[qb] <= kBigSum;
  }
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(!ok) != 0, 0)) {
    s_cur = scores32<D, NQ>(st, kc);
    rescale_half<D, NQ>(st, s_cur, sl2, acc);
    out = pack_half<NQ>(s_cur);
  }
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) st.l[qb] += acc[qb];
  return out;
}

// O^T += V^T P^T for one half, plain.
template <int D, int NQ>
__device__ __forceinline__ void pv_half(FwdState<D, NQ>& st, const __bf16* vt, const HalfP<NQ>& h) {
#pragma unroll
  for (int db = 0; db < D / 16; ++db) {
    const bf16x8 v = v_frag<D>(vt, db);
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) st.o[qb][db] = mfma16(v, h.p[qb], st.o[qb][db]);
  }
}

// Masked half for the ragged tails (keys >= nvalid are outside the span); always takes the
// exact path (row max, rescale when it grew), since tails are rare.
template <int D, int NQ>
__device__ __forceinline__ void masked_half(FwdState<D, NQ>& st, const __bf16* kt, const __bf16* vt, int nvalid,
                                            float sl2) {
  const int g = (threadIdx.x & 63) >> 4;
  HalfS<NQ> s = scores32<D, NQ>(st, kt);
#pragma unroll
  for (int j = 0; j < 2 * NQ; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) s.b[j][i] = (16 * (j / NQ) + 4 * g + i) < nvalid ? s.b[j][i] : -INFINITY;
  float sum[NQ];
  rescale_half<D, NQ>(st, s, sl2, sum);
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) st.l[qb] += sum[qb];
  pv_half<D, NQ>(st, vt, pack_half<NQ>(s));
}

template <int D, int NQ, int NS>
__global__ void __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
sra_fwd_kernel(FwdArgs a) {
  constexpr int NC = D / 32, ND = D / 16, BK = kFwdKeyStep, RK = kPadRS<D>, RV = kPadRS<D>;
  constexpr int KE = KTile<D>::kElems, VE = VTile<D>::kElems;
  // Three buffers each for K and V, as separate arrays addressed only with compile-time
  // choices (the loop is unrolled by three): the compiler can then tell a buffer being filled
  // by direct loads from the ones being read, and does not stall the reads on those loads.
  __shared__ __attribute__((aligned(1024))) __bf16 kbuf0[KE];
  __shared__ __attribute__((aligned(1024))) __bf16 kbuf1[KE];
  __shared__ __attribute__((aligned(1024))) __bf16 kbuf2[KE];
  __shared__ __attribute__((aligned(1024))) __bf16 vbuf0[VE];
  __shared__ __attribute__((aligned(1024))) __bf16 vbuf1[VE];
  __shared__ __attribute__((aligned(1024))) __bf16 vbuf2[VE];
  __bf16* const kb[3] = {kbuf0, kbuf1, kbuf2};
  __bf16* const vb[3] = {vbuf0, vbuf1, vbuf2};

  const WorkItem it = a.items[blockIdx.x];
  if (it.stream < 0) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, l16 = lane & 15;
  const int h = it.head, s = it.stream;
  const int wrow0 = wave * 16 * NQ;
  const bool active = wrow0 < it.len;
  const float sl2 = a.scale_log2;

  FwdState<D, NQ> st;
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    const int r = wrow0 + 16 * qb + l16;
    const __bf16* src = a.q[s] + int64_t(it.start + min(r, it.len - 1)) * a.in_stride[s] + h * D + g * 8;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const bf16x8 x = *reinterpret_cast<const bf16x8*>(src + c * 32);
      st.qf[qb][c] = (r < it.len) ? x : bf16x8{};
    }
#pragma unroll
    for (int db = 0; db < ND; ++db) st.o[qb][db] = floatx4{};
    st.m[qb] = -INFINITY;
    st.l[qb] = 0.f;
  }

  const Span* sp = a.spans + it.span_off;
  int T = 0;  // full tiles over all spans
  for (int i = 0; i < it.span_cnt; ++i) T += __builtin_amdgcn_readfirstlane(sp[i].len) / BK;

  // byte offsets of this wave's direct loads from the tile's first row (K and V tiles are laid
  // out alike; the streams differ in their token stride)
  using TL = PaddedTile<D, BK, RK>;
  constexpr int kSlots = (TL::kInstr + kWaves - 1) / kWaves, kFull = TL::kInstr / kWaves;
  uint32_t voff[NS][kSlots];
#pragma unroll
  for (int ss = 0; ss < NS; ++ss) {
    TileLoader<D, BK, RK, kWaves> tl;
    tl.init(a.in_stride[ss], h, wave);
#pragma unroll
    for (int j = 0; j < kSlots; ++j) voff[ss][j] = uint32_t(tl.voff[j]) * 2;
  }
  FullTileCursor<BK> kc, vc;  // next full tile to load for K, for V
  kc.init(sp, it.span_cnt);
  vc.init(sp, it.span_cnt);
  // per-stream bases as uniform scalars and this wave's LDS slots as byte addresses, so a
  // tile's loads need no argument reads and no address arithmetic per lane
  const uint64_t kb0 = uniform_u64(reinterpret_cast<uint64_t>(a.k[0]));
  const uint64_t kb1 = uniform_u64(reinterpret_cast<uint64_t>(a.k[1]));
  const uint64_t vb0 = uniform_u64(reinterpret_cast<uint64_t>(a.v[0]));
  const uint64_t vb1 = uniform_u64(reinterpret_cast<uint64_t>(a.v[1]));
  const int64_t st0 = a.in_stride[0] * 2, st1 = a.in_stride[1] * 2;  // bytes
  const bool extra = wave + kFull * kWaves < TL::kInstr;
  auto issue = [&](const FullTileCursor<BK>& c, uint64_t b0, uint64_t b1, const __bf16* dst) __attribute__((always_inline)) {
    const int ss = c.cur_stream;
    const uint64_t g = (ss ? b1 : b0) + uint64_t(int64_t(c.cur_start + c.off) * (ss ? st1 : st0));
    const uint32_t la = lds_addr(dst) + wave * 1024;
#pragma unroll
    for (int j = 0; j < kSlots; ++j)
      if (j < kFull || extra)
        lds_dma_x4_off(g, NS == 1 || !ss ? voff[0][j] : voff[NS - 1][j], la + j * kWaves * 1024);
  };
  auto issue_k = [&](const __bf16* dst) __attribute__((always_inline)) {
    issue(kc, kb0, kb1, dst);
    kc.advance();
  };
  auto issue_v = [&](const __bf16* dst) __attribute__((always_inline)) {
    issue(vc, vb0, vb1, dst);
    vc.advance();
  };

  // Pipelined full tiles. Tile t sits in K buffer t % 3 and V buffer t % 3 (tile -1 in V
  // buffer 2). Iteration t reads K(t) (second half), K(t+1) (first half), V(t-1) (second
  // half) and V(t) (first half), and loads K(t+2) and V(t+1).
  if (T > 0) {
    // V buffer 2 stands for tile -1: zero its second half so the first P V (P = 0) adds 0.
    for (int e = threadIdx.x * 8; e < 32 * RV; e += kWaves * 64 * 8)
      *reinterpret_cast<bf16x8*>(vbuf2 + 32 * RV + e) = bf16x8{};
    issue_k(kbuf0);
    issue_v(vbuf0);
    if (T > 1) issue_k(kbuf1);
    wait_vmem();
    __syncthreads();
    HalfP<NQ> p_hi;  // P of the previous tile's second half (zero before the first tile)
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) p_hi.p[qb] = bf16x8{};
    HalfS<NQ> s_lo = {}, s_hi = {};
    if (active) s_lo = scores32<D, NQ>(st, kbuf0);
    Ahead ah;
#pragma unroll
    for (int i = 0; i < kLook; ++i) {
      ah.k[i] = k_frag<D>(kbuf0 + 32 * RK, i);
      ah.v[i] = v_frag<D>(vbuf2 + 32 * RV, i);
    }
    auto iteration = [&](int t, auto phase) {
      constexpr int P = decltype(phase)::value;
      __bf16* const k_t = kb[P];
      __bf16* const k_t1 = kb[(P + 1) % 3];
      __bf16* const v_tm1 = vb[(P + 2) % 3];
      __bf16* const v_t = vb[P];
      if (t + 1 < T) issue_v(vb[(P + 1) % 3]);
      if (t + 2 < T) issue_k(kb[(P + 2) % 3]);
      if (active) {
        // block 1: S^T of this tile's second half and P V of the previous tile's second
        // half, under the softmax of this tile's first half
        const HalfP<NQ> p_lo = pipe_block<D, NQ>(st, s_lo, k_t, s_hi, k_t + 32 * RK, v_tm1 + 32 * RV, k_t1, v_t, ah, p_hi, sl2);
        // block 2: S^T of the next tile's first half and P V of this tile's first half,
        // under the softmax of this tile's second half (the last iteration's S^T is unused)
        p_hi = pipe_block<D, NQ>(st, s_hi, k_t + 32 * RK, s_lo, k_t1, v_t, k_t1 + 32 * RK, v_t + 32 * RV, ah, p_lo, sl2);
      }
      wait_vmem();
      __syncthreads();
    };
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using P2 = std::integral_constant<int, 2>;
    int t = 0;
    for (; t + 3 <= T; t += 3) {
      iteration(t, P0{});
      iteration(t + 1, P1{});
      iteration(t + 2, P2{});
    }
    if (t < T) iteration(t, P0{});
    if (t + 1 < T) iteration(t + 1, P1{});
    // the last tile's second half: V(T-1) sits in buffer (T-1) % 3
    if (active) {
      const int last = (T - 1) % 3;
      if (last == 0) pv_half<D, NQ>(st, vbuf0 + 32 * RV, p_hi);
      else if (last == 1) pv_half<D, NQ>(st, vbuf1 + 32 * RV, p_hi);
      else pv_half<D, NQ>(st, vbuf2 + 32 * RV, p_hi);
    }
  }

  // Ragged span tails (masked, not pipelined).
  for (int i = 0; i < it.span_cnt; ++i) {
    const Span sp_i = sp[i];
    const int len = __builtin_amdgcn_readfirstlane(sp_i.len);
    const int rem = len % BK;
    if (rem == 0) continue;
    __syncthreads();  // every wave is done with the buffers
    const int ss = __builtin_amdgcn_readfirstlane(sp_i.stream);
    const int st0 = __builtin_amdgcn_readfirstlane(sp_i.start);
    tile_load_lds<D, BK, RK, kWaves>(kbuf0, a.k[ss], a.in_stride[ss], h, st0, len, len - rem, wave);
    tile_load_lds<D, BK, RV, kWaves>(vbuf0, a.v[ss], a.in_stride[ss], h, st0, len, len - rem, wave);
    wait_vmem();
    __syncthreads();
    if (active) {
      masked_half<D, NQ>(st, kbuf0, vbuf0, rem, sl2);
      if (rem > 32) masked_half<D, NQ>(st, kbuf0 + 32 * RK, vbuf0 + 32 * RV, rem - 32, sl2);
    }
  }

  if (!active) return;
  const int64_t ostride = int64_t(a.heads) * D;
  float* part = it.slot ? a.part + int64_t(it.slot - 1) * (kWaves * 16 * NQ) * (D + 2) : nullptr;
#pragma unroll
  for (int qb = 0; qb < NQ; ++qb) {
    const int r = wrow0 + 16 * qb + l16;
    const float lt = quad_sum(st.l[qb]);
    if (part) {  // a piece of a split item
      if (r >= it.len) continue;
#pragma unroll
      for (int db = 0; db < ND; ++db) *reinterpret_cast<floatx4*>(part + r * D + db * 16 + 4 * g) = st.o[qb][db];
      if (g == 0) *reinterpret_cast<float2*>(part + kWaves * 16 * NQ * D + 2 * r) = float2{st.m[qb], lt};
      continue;
    }
    const float inv = 1.f / lt;
    if (r >= it.len) continue;
    __bf16* orow = a.o[s] + int64_t(it.start + r) * ostride + h * D;
#pragma unroll
    for (int db = 0; db < ND; ++db) {
      bf16x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = (__bf16)(st.o[qb][db][e] * inv);
      *reinterpret_cast<bf16x4*>(orow + db * 16 + 4 * g) = w;
    }
    if (g == 0) a.lse[s][int64_t(h) * a.rows[s] + it.start + r] = (st.m[qb] + log2f(lt)) * kLn2;
  }
}

// Rows of the split items from their pieces: with M the largest of the pieces' running maxima,
// O = sum_i 2^(m_i - M) O_i / sum_i 2^(m_i - M) l_i, in piece order. D / 4 threads per row. A piece whose
// scores of a row are all -inf has weight 0; a row of which all are so ends as in a whole item (LSE -inf).
// Bound by reading the partial results (28 MB at most): 3 heads of 800 + 429 tokens 38.5 -> 25.3 us.
template <int D>
__global__ void __launch_bounds__(kThreads) sra_fwd_combine_kernel(FwdArgs a, const CombineItem* items) {
  constexpr int TPR = D / 4, RPB = kThreads / TPR;
  const CombineItem it = items[blockIdx.x];
  const int r = blockIdx.y * RPB + threadIdx.x / TPR, sub = threadIdx.x % TPR, tile = a.tile;
  if (r >= it.len) return;
  const int64_t slot = int64_t(tile) * (D + 2);
  const float* p = a.part + it.slot0 * slot;
  float m = -INFINITY;
  for (int i = 0; i < it.n; ++i) m = fmaxf(m, p[i * slot + int64_t(tile) * D + 2 * r]);
  floatx4 o = floatx4{};
  float l = 0.f;
  for (int i = 0; i < it.n; ++i) {
    const float2 ml = *reinterpret_cast<const float2*>(p + i * slot + int64_t(tile) * D + 2 * r);
    const float w = ml.x == -INFINITY ? 0.f : fast_exp2(ml.x - m);
    l += w * ml.y;
    o += w * *reinterpret_cast<const floatx4*>(p + i * slot + r * D + 4 * sub);
  }
  const float inv = 1.f / l;
  bf16x4 y;
#pragma unroll
  for (int e = 0; e < 4; ++e) y[e] = (__bf16)(o[e] * inv);
  *reinterpret_cast<bf16x4*>(a.o[it.stream] + (int64_t(it.start + r) * a.heads + it.head) * D + 4 * sub) = y;
  if (sub == 0) a.lse[it.stream][int64_t(it.head) * a.rows[it.stream] + it.start + r] = (m + log2f(l)) * kLn2;
}

template <int D, int NQ>
static void launch_tile(const FwdArgs& a, int n_items, hipStream_t stream) {
  const dim3 grid(n_items), block(kWaves * 64);
  if (a.in_stride[0] == a.in_stride[1])
    hipLaunchKernelGGL((sra_fwd_kernel<D, NQ, 1>), grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((sra_fwd_kernel<D, NQ, 2>), grid, block, 0, stream, a);
}

hipError_t launch_forward(const FwdArgs& a, int n_items, int head_dim, bool mfma32, hipStream_t stream) {
  if (n_items <= 0) return hipSuccess;
  if (mfma32) return launch_forward32(a, n_items, head_dim, stream);
  if (head_dim == 64) launch_tile<64, fwd_large_tile(64) / 128>(a, n_items, stream);
  else if (a.tile == kFwdQueryTile) launch_tile<128, kFwdQueryTile / 128>(a, n_items, stream);
  else launch_tile<128, fwd_large_tile(128) / 128>(a, n_items, stream);
  return hipGetLastError();
}

hipError_t launch_forward_combine(const FwdArgs& a, const CombineItem* items, int n, int head_dim, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const int rows = kThreads / (head_dim / 4);
  const dim3 grid(n, (a.tile + rows - 1) / rows);
  if (head_dim == 128)
    hipLaunchKernelGGL(sra_fwd_combine_kernel<128>, grid, dim3(kThreads), 0, stream, a, items);
  else
    hipLaunchKernelGGL(sra_fwd_combine_kernel<64>, grid, dim3(kThreads), 0, stream, a, items);
  return hipGetLastError();
}

}  // namespace sra
