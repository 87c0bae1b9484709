// Tile shapes and schedule records shared by the host scheduler and the HIP kernels.
#pragma once
#include <stdint.h>

namespace sra {

// Forward: one workgroup = 8 wave64s (two per SIMD), each wave owns 32 query rows, so a work
// item covers 256 query rows; keys stream through LDS 64 at a time. Long calls run with more rows
// per wave (as many as its registers hold: 48 at d = 128, 64 at d = 64), which read and load the
// keys less often.
constexpr int kFwdQueryTile = 256;
constexpr int kFwdKeyStep = 64;
constexpr int fwd_large_tile(int head_dim) { return head_dim == 128 ? 384 : 512; }
// dQ kernel of the backward: 256-row query tiles, held by 4 wave64s (one per
// SIMD, 64 query rows each); keys stream through LDS 64 at a time. kDqKeyStep and kDkvQueryStep
// are the steps in which the whole schedules of the inspection hooks count phases; what is launched
// counts them in kStep.
constexpr int kDqQueryTile = 256;
constexpr int kDqKeyStep = 32;
// dK/dV kernel of the backward: 4 wave64s (one per SIMD) x 64 keys = 256 keys per work item;
// queries stream through LDS 64 at a time.
constexpr int kDkvKeyTile = 256;
constexpr int kDkvQueryStep = 32;

constexpr int kThreads = 256;  // block size of the element-wise kernels (delta, fill, gather, scatter)
constexpr int kNumXcd = 8;  // MI355X: 8 accelerator complex dies; workgroups go round-robin
constexpr int kCusPerXcd = 32;  // 256 compute units
constexpr int kNumCus = kNumXcd * kCusPerXcd;
constexpr int kStep = 64;  // rows of an LDS tile: where a work item's spans can be cut

// One work item: a tile of rows of one stream and head, and the list of row ranges of the
// other side it pairs with (key spans for query tiles, query spans for key tiles).
struct WorkItem {
  int32_t stream;      // 0 = generation, 1 = reference, -1 = padding (no work)
  int32_t head;
  int32_t start;       // first packed token row of the tile
  int32_t len;         // rows in the tile (<= tile size)
  int32_t span_off;    // first entry in the span table
  int32_t span_cnt;
  int32_t sample;
  int32_t slot;        // 0: the item's results are final; k > 0: one piece of a split item, whose
                       // fp32 partial results go to slot k - 1 of the launch's scratch
};

// A work item split into n pieces (each over a part of its spans, slots slot0 ..): the combine
// kernels add the partial results up in piece order.
struct CombineItem {
  int32_t stream;
  int32_t head;
  int32_t start;
  int32_t len;
  int32_t slot0;
  int32_t n;
  int32_t reserved[2];
};

struct Span {
  int32_t stream;      // 0 = generation, 1 = reference
  int32_t start;       // first packed token row
  int32_t len;         // rows (> 0)
  int32_t keys;        // key-major schedules: the work item's keys [lo, hi) (tile-relative) this
                       // span reaches, packed lo | hi << 16; 0 = every key of the item
};

// Row range of a stream whose outputs are constant (invalid reference frames).
struct FillRange {
  int32_t stream;
  int32_t start;
  int32_t len;
  int32_t reserved;
};

}  // namespace sra
