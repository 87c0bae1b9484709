// Direct global -> LDS staging of padded [rows x D] bf16 tiles and the span walk of the kernels.
#pragma once
#include "sra_config.h"
#include "sra_device.h"

namespace sra {

// Padded LDS tiles: NR rows of D bf16 with a row stride of RS elements, so every fragment
// address is one per-lane base plus a compile-time offset. The operands of 16x16x32 MFMAs read
// rows of 16 (row fragments by ds_read_b128: 16 rows x 64 bytes, lanes {0-3, 12-15, 20-27} and
// so on served together; transpose reads by ds_read_b64_tr_b16: 8 rows x 32 bytes served
// together): a stride of D + 16 serves both without bank conflicts (measured 4.5 and 2.6 cycles
// per wave read; D + 8 takes 8.2 and 4.3, D + 24 8.2 and 4.3).
template <int D> constexpr int kPadRS = D + 16;
// 32x32x16 MFMAs take 32 rows per fragment: row fragments of 32 rows x 32 bytes and transpose reads of
// 4 rows x 4 chunks, both at 128 bytes per clock with a stride of D + 8 and, for the transpose
// reads, the rows of each block of 16 permuted: logical row r = 4a + b (a, b < 4) sits at physical
// row 4b + a. The map is its own inverse, and for r < 8 it sends r + 8 to perm16(r) + 2.
template <int D> constexpr int kPadRS32 = D + 8;
__host__ __device__ constexpr int perm16(int r) { return (r & ~15) | ((r & 3) << 2) | ((r >> 2) & 3); }

template <int D, int NR, int RS>
struct PaddedTile {
  static constexpr int kSlotsPerRow = RS / 8;                          // 16-byte slots per row
  static constexpr int kInstr = (NR * kSlotsPerRow + 63) / 64;         // 1 KB load instructions
  static constexpr int kElems = kInstr * 512;                          // LDS elements to reserve
};

// One GLOBAL_LOAD_LDS_DWORDX4: lane l copies 16 bytes from g to (lds + 16 l); lds is uniform.
// Issued as inline assembly on purpose: the compiler then does not see an LDS write in
// flight, and does not stall the LDS reads of the other buffers (which it cannot prove
// disjoint) until the copy lands. Every reader of a buffer filled this way waits with
// wait_vmem() and a workgroup barrier first. M0 holds the LDS address for the copy; it is
// reserved by the compiler, so it is restored right after the instruction has read it.
__device__ __forceinline__ void lds_dma_x4(const void* g, void* lds) {
  const uint32_t la = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)lds);
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "v"(g), "s"(la)
      : "memory");
}

// A wave-uniform 64-bit value held in scalar registers.
__device__ __forceinline__ uint64_t uniform_u64(uint64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(x));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(x >> 32));
  return (uint64_t(hi) << 32) | lo;
}

// LDS byte address of a __shared__ object.
template <class T>
__device__ __forceinline__ uint32_t lds_addr(const T* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// lds_dma_x4 to an LDS byte address (uniform) computed by the caller.
__device__ __forceinline__ void lds_dma_x4_at(const void* g, uint32_t la) {
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "v"(g), "s"(__builtin_amdgcn_readfirstlane(la))
      : "memory");
}

// The same with a uniform global base and a 32-bit byte offset per lane.
__device__ __forceinline__ void lds_dma_x4_off(uint64_t base, uint32_t off, uint32_t la) {
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %3\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, %2\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "v"(off), "s"(base), "s"(la)
      : "memory");
}

// Swizzled LDS tiles: NR rows of D bf16 without padding, the 16-byte chunks of row r XORed with
// swz<D>(r). Both reads of the 16x16x32 MFMA operands are then free of bank conflicts (row
// fragments by ds_read_b128, whose lanes {0-3, 12-15, 20-27} are served together, and transpose
// reads, served 32 lanes at a time: 4.5 and 2.6 cycles per wave read measured, against 8.1 and
// 4.3 with two-way conflicts), and a tile is a whole number of 1 KB loads.
template <int D>
__host__ __device__ constexpr int swz(int r) {
  return D == 128 ? 2 * (r & 7) : 2 * ((r >> 1) & 3);
}
template <int D, int NR>
struct SwzTile {
  static constexpr int kInstr = NR * D / 512;    // 1 KB load instructions
  static constexpr int kElems = NR * D;
  static constexpr int kRowsPerInstr = 512 / D;
};
// Byte address of this lane's part of row fragment c = 0 (rows 0..15, head dims 0..31); fragment c
// is at the address XOR 64 c, rows 16 n further at + 32 n D.
template <int D>
__device__ __forceinline__ uint32_t swz_row_addr() {
  const int lane = threadIdx.x & 63, r = lane & 15;
  return uint32_t(r * D * 2 + (((lane >> 4) ^ swz<D>(r)) * 16));
}
// The same for the transpose reads of a 16-row x 16-dim block (lane group g holds rows 4 g .. + 3):
// head dims 16 db .. + 15 are at the address XOR 32 db.
template <int D>
__device__ __forceinline__ uint32_t swz_tr_addr() {
  const int lane = threadIdx.x & 63, r = 4 * (lane >> 4) + ((lane & 15) >> 2);
  return uint32_t(r * D * 2 + ((((lane & 3) >> 1) ^ swz<D>(r)) * 16) + (lane & 1) * 8);
}
// a XOR a constant, computed where it stands: left to the compiler, the addresses of a phase's
// fragments are all computed ahead of it and hold a register each.
template <int K>
__device__ __forceinline__ uint32_t xor_here(uint32_t a) {
  if constexpr (K == 0) return a;
  uint32_t r;
  asm volatile("v_xor_b32 %0, %2, %1" : "=v"(r) : "v"(a), "i"(K));
  return r;
}
__device__ __forceinline__ bf16x8 lds_ld8(uint32_t a) {
  return *(const __attribute__((address_space(3))) bf16x8*)(uintptr_t)a;
}
__device__ __forceinline__ floatx4 lds_ld4f(uint32_t a) {
  return *(const __attribute__((address_space(3))) floatx4*)(uintptr_t)a;
}
__device__ __forceinline__ void lds_st_f(uint32_t a, float x) {
  *(__attribute__((address_space(3))) float*)(uintptr_t)a = x;
}
__device__ __forceinline__ bf16x4 lds_ld_tr(uint32_t a) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(uintptr_t)a);
}
// Byte offset of this lane's chunk of load instruction `wave` of a swizzled tile from the tile's
// first row (the instructions of a wave are a multiple of 4 apart, so they share it up to a
// whole number of rows).
template <int D>
__device__ __forceinline__ uint32_t swz_load_off(int64_t stride, int head, int wave) {
  constexpr int CPR = D / 8;
  const int lane = threadIdx.x & 63, r = wave * (512 / D) + lane / CPR;
  return uint32_t((int64_t(r) * stride + head * D + ((lane % CPR) ^ swz<D>(r)) * 8) * 2);
}
// Rows [off, off + NR) of a span into a swizzled tile, rows past the span's end clamped to its last.
template <int D, int NR, int NW>
__device__ __forceinline__ void swz_load_clamped(uint32_t la, uint64_t src, int64_t stride, int head, int start, int len,
                                                 int off, int wave) {
  constexpr int CPR = D / 8, RPI = 512 / D;
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < SwzTile<D, NR>::kInstr / NW; ++j) {
    const int r = (wave + j * NW) * RPI + lane / CPR;
    const int rr = min(off + r, len - 1);
    const __bf16* g = reinterpret_cast<const __bf16*>(src) + int64_t(start + rr) * stride + head * D +
                      ((lane % CPR) ^ swz<D>(r)) * 8;
    lds_dma_x4_at(g, la + (wave + j * NW) * 1024);
  }
}

// The same for 4 bytes per lane (lane l's land at la + 4 l).
__device__ __forceinline__ void lds_dma_x1_off(uint64_t base, uint32_t off, uint32_t la) {
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %3\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dword %1, %2\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "v"(off), "s"(base), "s"(la)
      : "memory");
}

// Direct global -> LDS copy (gfx950 GLOBAL_LOAD_LDS_DWORDX4) of rows [off, off + NR) of a span
// into a padded tile. Each wave instruction fills 1 KB of LDS: lane l writes the 16 bytes at
// (LDS base + 16 l), so lane l fetches the global chunk that belongs there; lanes that land on
// a pad slot fetch an in-bounds chunk that nothing reads. Rows past the span end are clamped
// to its last row (the kernels mask them). Instructions are dealt over the NW waves. kPerm: rows
// permuted in blocks of 16 (perm16).
template <int D, int NR, int RS, int NW, bool kPerm = false>
__device__ __forceinline__ void tile_load_lds(__bf16* lds, const __bf16* __restrict__ src, int64_t stride,
                                              int head, int start, int len, int off, int wave) {
  using TL = PaddedTile<D, NR, RS>;
  constexpr int SPR = TL::kSlotsPerRow, CPR = D / 8;
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < (TL::kInstr + NW - 1) / NW; ++j) {
    const int ins = wave + j * NW;
    if (ins < TL::kInstr) {
      const int p = ins * 64 + lane;
      const int prow = min(p / SPR, NR - 1);
      const int row = kPerm ? perm16(prow) : prow;
      const int slot = p % SPR;
      const int ch = slot < CPR ? slot : 0;
      const int rr = min(off + row, len - 1);
      const __bf16* g = src + int64_t(start + rr) * stride + head * D + ch * 8;
      lds_dma_x4(g, lds + ins * 512);
    }
  }
}

// Per-lane address offsets of the direct loads of a padded tile, for tiles whose NR rows all
// lie inside the span (no clamping): lane offsets are fixed, only the tile's first row moves.
template <int D, int NR, int RS, int NW, bool kPerm = false>
struct TileLoader {
  using TL = PaddedTile<D, NR, RS>;
  static constexpr int kSlots = (TL::kInstr + NW - 1) / NW;
  int voff[kSlots];  // element offset of this lane's chunk from the tile's first row
  __device__ __forceinline__ void init(int64_t stride, int head, int wave) {
    constexpr int SPR = TL::kSlotsPerRow, CPR = D / 8;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
      const int p = (wave + j * NW) * 64 + lane;
      const int prow = min(p / SPR, NR - 1);
      const int row = kPerm ? perm16(prow) : prow;
      const int slot = p % SPR;
      voff[j] = int(row * stride) + head * D + (slot < CPR ? slot : 0) * 8;
    }
  }
};

__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A workgroup barrier that waits for nothing else: LDS reads and direct loads in flight stay so
// (__syncthreads waits for all of them). The caller has waited for the loads that are read next.
__device__ __forceinline__ void block_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Walks the full STEP-row tiles of a span list (ragged span ends are skipped).
template <int STEP>
struct FullTileCursor {
  const Span* spans;
  int n, si, off, cur_stream, cur_start, cur_len;
  __device__ __forceinline__ void settle() {
    while (si < n) {
      const Span s = spans[si];
      cur_stream = __builtin_amdgcn_readfirstlane(s.stream);
      cur_start = __builtin_amdgcn_readfirstlane(s.start);
      cur_len = __builtin_amdgcn_readfirstlane(s.len);
      if (off + STEP <= cur_len) return;
      ++si;
      off = 0;
    }
  }
  __device__ __forceinline__ void init(const Span* s, int count) {
    spans = s;
    n = count;
    si = 0;
    off = 0;
    settle();
  }
  __device__ __forceinline__ void advance() {
    off += STEP;
    if (off + STEP > cur_len) {
      ++si;
      off = 0;
      settle();
    }
  }
};

}  // namespace sra
