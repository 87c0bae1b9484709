// Geometry -> visibility runs -> tile schedules (host).
//
// Visibility (Avatar V §1, §2.1, §4.3, §8): a gen query sees every gen key of its sample and
// every valid ref key of its sample; a valid ref query sees the valid ref keys of its own
// group of `group_frames` frames. A ref token is valid when its frame is and, if the sample
// carries a token mask, its own entry is (§4.3 invalid tokens). The rule is expressed here
// as contiguous row ranges ("spans") built from the runs of valid ref rows, so each work
// item's kernel loop visits only visible key (or query) rows and masks nothing but the
// ragged end of a span and, in the key-major schedule, the keys of a tile that a group's
// reference queries do not reach.
#include "schedule.hpp"

#include <algorithm>
#include <cmath>
#include <map>
#include <queue>
#include <cstdio>
#include <numeric>

namespace sra {

namespace {

struct Run {  // [f0, f1) frames
  int32_t f0, f1;
};

struct RowRun {  // [r0, r1) ref rows (sample-relative), all valid
  int64_t r0, r1;
};

// Maximal runs of valid ref rows inside [lo, hi).
std::vector<RowRun> valid_runs(const SampleLayout& s, int64_t lo, int64_t hi) {
  std::vector<RowRun> runs;
  for (const auto& r : s.vruns) {
    const int64_t a = std::max(lo, r.first), b = std::min(hi, r.second);
    if (a < b) runs.push_back({a, b});
  }
  return runs;
}

// Rows of ref group g0 (its first frame) of a sample.
RowRun group_rows(const SampleLayout& s, int32_t g0) {
  if (!s.gbound.empty()) return {s.gbound[g0 / s.group], s.gbound[g0 / s.group + 1]};
  return {int64_t(g0) * s.F, int64_t(std::min(s.ref_frames, g0 + s.group)) * s.F};
}

// Gen frames [f0, f1) a gen frame t sees under the sample's temporal window.
Run gen_window_frames(const SampleLayout& s, int32_t t) {
  return {std::max<int32_t>(0, t - s.window), std::min<int32_t>(s.gen_frames, t + s.window + 1)};
}

bool mul_ok(int64_t a, int64_t b, int64_t lim) { return a >= 0 && b >= 0 && (b == 0 || a <= lim / b); }

}  // namespace

sra_status make_layout(const sra_problem* p, Layout* out, std::string* err) {
  if (!p) { *err = "problem is NULL"; return SRA_ERR_INVALID_ARGUMENT; }
  if (p->batch < 1) { *err = "batch must be >= 1"; return SRA_ERR_INVALID_ARGUMENT; }
  if (p->num_heads < 1) { *err = "num_heads must be >= 1"; return SRA_ERR_INVALID_ARGUMENT; }
  if (p->head_dim != 64 && p->head_dim != 128) {
    *err = "head_dim " + std::to_string(p->head_dim) + " unsupported (64 or 128)";
    return p->head_dim > 0 ? SRA_ERR_UNSUPPORTED : SRA_ERR_INVALID_ARGUMENT;
  }
  if (!p->samples) { *err = "samples is NULL"; return SRA_ERR_INVALID_ARGUMENT; }
  if (p->flags & ~uint32_t(SRA_FLAG_GEN_QUERIES_ONLY | SRA_FLAG_GEN_WINDOW)) {
    *err = "unknown flag bits";
    return SRA_ERR_INVALID_ARGUMENT;
  }
  const bool windowed = (p->flags & SRA_FLAG_GEN_WINDOW) != 0;
  if (!(std::isfinite(p->softmax_scale))) { *err = "softmax_scale is not finite"; return SRA_ERR_INVALID_ARGUMENT; }
  const int64_t hd = int64_t(p->num_heads) * p->head_dim;
  Layout L;
  L.batch = p->batch;
  L.heads = p->num_heads;
  L.head_dim = p->head_dim;
  L.gen_only = (p->flags & SRA_FLAG_GEN_QUERIES_ONLY) != 0;
  L.scale = p->softmax_scale > 0.f ? p->softmax_scale : float(1.0 / std::sqrt(double(p->head_dim)));
  L.gen_stride = p->gen_token_stride == 0 ? hd : p->gen_token_stride;
  L.ref_stride = p->ref_token_stride == 0 ? hd : p->ref_token_stride;
  if (L.gen_stride < hd || L.ref_stride < hd) {
    *err = "token stride must be >= num_heads*head_dim";
    return SRA_ERR_INVALID_ARGUMENT;
  }
  const int64_t kRowLimit = (int64_t(1) << 31) - 1;
  // The kernels' tile loaders hold the offset of a row inside a tile (up to 63 rows past the
  // tile's first row, plus the head's columns) in 32 bits.
  if (L.gen_stride > kRowLimit / 64 || L.ref_stride > kRowLimit / 64) {
    *err = "token stride exceeds (2^31 - 1) / 64 elements (32-bit offsets inside a tile)";
    return SRA_ERR_UNSUPPORTED;
  }
  L.samples.resize(p->batch);
  for (int32_t b = 0; b < p->batch; ++b) {
    const sra_sample_geom& g = p->samples[b];
    SampleLayout& s = L.samples[b];
    const std::string tag = "sample " + std::to_string(b) + ": ";
    if (g.gen_frames < 1 || g.gen_h < 1 || g.gen_w < 1) {
      *err = tag + "generation frames/height/width must be >= 1";
      return SRA_ERR_INVALID_ARGUMENT;
    }
    if (g.ref_frames < 0 || g.ref_h < 0 || g.ref_w < 0 || (g.ref_frames > 0 && (g.ref_h < 1 || g.ref_w < 1))) {
      *err = tag + "reference frames must be >= 0 and height/width >= 1 when frames > 0";
      return SRA_ERR_INVALID_ARGUMENT;
    }
    if (g.group_frames < 1) { *err = tag + "group_frames must be >= 1"; return SRA_ERR_INVALID_ARGUMENT; }
    if (windowed && g.gen_window < 0) { *err = tag + "gen_window must be >= 0"; return SRA_ERR_INVALID_ARGUMENT; }
    if (!mul_ok(g.gen_frames, int64_t(g.gen_h) * g.gen_w, kRowLimit) ||
        !mul_ok(g.ref_frames, int64_t(g.ref_h) * g.ref_w, kRowLimit)) {
      *err = tag + "token count overflows int32";
      return SRA_ERR_INVALID_ARGUMENT;
    }
    s.G = int64_t(g.gen_frames) * g.gen_h * g.gen_w;
    s.Fg = int64_t(g.gen_h) * g.gen_w;
    s.gen_frames = g.gen_frames;
    // a window reaching every frame is no window (same schedule as full attention)
    s.window = (windowed && g.gen_window < g.gen_frames - 1) ? g.gen_window : -1;
    s.F = g.ref_frames > 0 ? int64_t(g.ref_h) * g.ref_w : 0;
    s.R = int64_t(g.ref_frames) * s.F;
    s.ref_frames = g.ref_frames;
    s.group = g.group_frames;
    // runs of valid ref rows from the frame mask and the token mask
    s.vruns.clear();
    int64_t open = -1;  // first row of the run being extended, -1 = none
    for (int32_t f = 0; f < g.ref_frames; ++f) {
      const bool fv = !g.ref_frame_valid || g.ref_frame_valid[f];
      if (!g.ref_token_valid) {  // a frame mask alone: whole frames open or close a run
        const int64_t r = int64_t(f) * s.F;
        if (fv && open < 0) open = r;
        if (!fv && open >= 0) {
          s.vruns.push_back({open, r});
          open = -1;
        }
        continue;
      }
      for (int64_t j = 0; j < s.F; ++j) {
        const int64_t r = int64_t(f) * s.F + j;
        const bool tv = fv && g.ref_token_valid[r];
        if (tv && open < 0) open = r;
        if (!tv && open >= 0) {
          s.vruns.push_back({open, r});
          open = -1;
        }
      }
    }
    if (open >= 0) s.vruns.push_back({open, s.R});
    s.gen_off = L.sum_gen;
    s.ref_off = L.sum_ref;
    L.sum_gen += s.G;
    L.sum_ref += s.R;
    if (L.sum_gen > kRowLimit || L.sum_ref > kRowLimit) {
      *err = "packed token count overflows int32";
      return SRA_ERR_INVALID_ARGUMENT;
    }
  }
  // The kernels index per-row statistics (log-sum-exp, -rowsum(dO * O)) as head * rows + row
  // and whole token rows as heads * head_dim elements, both in 32 bits.
  if (hd > kRowLimit || int64_t(L.heads) * std::max(L.sum_gen, L.sum_ref) > kRowLimit) {
    *err = "num_heads * packed tokens of a stream (or num_heads * head_dim) exceeds 2^31 - 1";
    return SRA_ERR_UNSUPPORTED;
  }
  *out = std::move(L);
  return SRA_OK;
}

void closed_form_pairs(const Layout& L, int64_t* gen_pairs, int64_t* ref_pairs) {
  int64_t gp = 0, rp = 0;
  for (const SampleLayout& s : L.samples) {
    int64_t valid_rows = 0;
    for (const auto& r : s.vruns) valid_rows += r.second - r.first;
    gp += s.G * valid_rows;
    if (s.window < 0) {
      gp += s.G * s.G;
    } else {
      for (int32_t t = 0; t < s.gen_frames; ++t) {
        const Run w = gen_window_frames(s, t);
        gp += s.Fg * s.Fg * (w.f1 - w.f0);
      }
    }
    for (int32_t g0 = 0; g0 < s.ref_frames; g0 += s.group) {
      const RowRun gr = group_rows(s, g0);
      int64_t n = 0;
      for (const RowRun& r : valid_runs(s, gr.r0, gr.r1)) n += r.r1 - r.r0;
      rp += n * n;
    }
  }
  if (gen_pairs) *gen_pairs = gp;
  if (ref_pairs) *ref_pairs = L.gen_only ? 0 : rp;
}

namespace {

struct TileClass {   // tiles sharing one span list
  int32_t stream;
  int64_t row0, rows;            // packed rows covered (tiled)
  int32_t span_off, span_cnt;
  int32_t sample;
  int64_t other_rows;            // total rows over the span list
};

// Tiles rows [row0, row0+rows) of `stream` with `tile` rows each; one item per tile and head.
void emit_items(const TileClass& c, int tile, int32_t heads, int step,
                const std::vector<Span>& spans, std::vector<std::pair<int64_t, WorkItem>>* out) {
  int64_t step_rows = 0;  // work estimate: span rows rounded up to the inner step
  for (int32_t i = 0; i < c.span_cnt; ++i) {
    int64_t l = spans[c.span_off + i].len;
    step_rows += (l + step - 1) / step * step;
  }
  for (int32_t h = 0; h < heads; ++h)
    for (int64_t r = 0; r < c.rows; r += tile) {
      WorkItem w;
      w.stream = c.stream;
      w.head = h;
      w.start = int32_t(c.row0 + r);
      w.len = int32_t(std::min<int64_t>(tile, c.rows - r));
      w.span_off = c.span_off;
      w.span_cnt = c.span_cnt;
      w.sample = c.sample;
      w.slot = 0;
      out->push_back({int64_t(tile) * step_rows, w});
    }
}

void longest_first(std::vector<std::pair<int64_t, WorkItem>>& v) {
  const auto longer = [](const auto& a, const auto& b) { return a.first > b.first; };
  if (!std::is_sorted(v.begin(), v.end(), longer)) std::stable_sort(v.begin(), v.end(), longer);
}

// Lists items in launch order. Workgroups are dealt round-robin over the 8 XCDs, so item k of
// the launch order runs on XCD k % 8 and each XCD consumes its own subsequence in order.
// When heads divide evenly over the XCDs, every head is pinned to one XCD (the rows it streams
// stay in that XCD's L2), whose subsequence holds its items in v's order; otherwise the
// round-robin deal of v balances it.
void deal_items(const std::vector<WorkItem>& v, int32_t heads, Schedule* s) {
  s->real_items = int64_t(v.size());
  s->items.clear();
  if (heads % kNumXcd != 0) {
    s->items = v;
    return;
  }
  std::vector<std::vector<WorkItem>> per(kNumXcd);
  for (auto& q : per) q.reserve(v.size() / kNumXcd + 1);
  for (const WorkItem& w : v) per[w.head % kNumXcd].push_back(w);
  size_t n = 0;
  for (auto& q : per) n = std::max(n, q.size());
  WorkItem pad{};
  pad.stream = -1;
  s->items.reserve(n * kNumXcd);
  for (size_t j = 0; j < n; ++j)
    for (int x = 0; x < kNumXcd; ++x) s->items.push_back(j < per[x].size() ? per[x][j] : pad);
}

// Orders items for launch, longest first.
// heads_in_turn: each XCD runs its heads one after another instead, each head's items
// longest-first. For key tiles, whose items are of a few similar lengths and all stream the
// head's gen queries from the first row, this keeps the workgroups resident on an XCD on one
// head and close together in its query stream (measured at 720p: half the L2 misses, 1.5 %
// faster). Query tiles keep the plain order: there the long gen tiles of all the XCD's heads
// run back to back in step, and putting each head's short ref tiles between them staggered
// the next head's start and nearly tripled the misses.
void order_items(std::vector<std::pair<int64_t, WorkItem>>& v, int32_t heads, bool heads_in_turn, Schedule* s) {
  longest_first(v);
  std::vector<WorkItem> w;
  w.reserve(v.size());
  for (auto& e : v) w.push_back(e.second);
  if (heads_in_turn && heads % kNumXcd == 0)
    std::stable_sort(w.begin(), w.end(), [](const WorkItem& a, const WorkItem& b) { return a.head < b.head; });
  deal_items(w, heads, s);
}

// Phase alignment of a schedule (runs after order_items with heads pinned to XCDs). The first
// span of a key tile is the sample's gen query rows, and that of a gen query tile the sample's
// gen keys: every such tile of a sample and head streams the same rows, and the tiles resident
// on an XCD share them through its L2 only while they are at nearby steps of the span at the
// same time. Tiles start whenever a compute unit frees up, so tiles of different lengths drift
// apart. Here each XCD's launch order is replayed on its compute units (one resident tile
// each, time counted in steps of `step` rows: in what is launched the LDS tile of the kernels, so
// that a span is cut where a tile ends): a tile predicted to start at time t begins its first span
// at step t mod S (S = the span's steps) and wraps around, so that all tiles stream step t mod S
// at time t. The tile's pairs are unchanged (the span is cut in two); only
// the order of the sums changes, fixed by the plan.
void align_phases(int step, Schedule* s) {
  std::vector<Span> spans;
  std::map<std::pair<int32_t, int32_t>, int32_t> made;  // (span list, phase in rows) -> offset
  const size_t n = s->items.size();
  for (int x = 0; x < kNumXcd; ++x) {
    std::priority_queue<int64_t, std::vector<int64_t>, std::greater<int64_t>> free_at;
    for (int c = 0; c < kCusPerXcd; ++c) free_at.push(0);
    for (size_t k = size_t(x); k < n; k += kNumXcd) {
      WorkItem& w = s->items[k];
      if (w.stream < 0 || w.span_cnt <= 0) continue;
      const Span* l = &s->spans[size_t(w.span_off)];
      int64_t cost = 0;
      for (int32_t i = 0; i < w.span_cnt; ++i) cost += (l[i].len + step - 1) / step;
      const int64_t t0 = free_at.top();
      free_at.pop();
      free_at.push(t0 + cost);
      const int64_t first_steps = (l[0].len + step - 1) / step;
      int32_t phase = 0;
      if (l[0].stream == 0 && l[0].keys == 0 && first_steps > 1) phase = int32_t(t0 % first_steps) * step;
      const auto key = std::make_pair(w.span_off, phase);
      auto it = made.find(key);
      if (it == made.end()) {
        const int32_t off = int32_t(spans.size());
        if (phase == 0) {
          spans.push_back(l[0]);
        } else {
          spans.push_back({l[0].stream, l[0].start + phase, l[0].len - phase, 0});
          spans.push_back({l[0].stream, l[0].start, phase, 0});
        }
        spans.insert(spans.end(), l + 1, l + w.span_cnt);
        it = made.emplace(key, off).first;
      }
      w.span_cnt += phase == 0 ? 0 : 1;
      w.span_off = it->second;
    }
  }
  s->spans.swap(spans);
}

typedef std::vector<std::pair<int64_t, WorkItem>> CostedItems;

// Query-major items (forward and dQ): query tiles of `tile` rows, key spans per class.
CostedItems query_major_items(const Layout& L, int tile, int step, Schedule* s) {
  std::vector<TileClass> classes;
  s->spans.clear();
  for (int32_t b = 0; b < L.batch; ++b) {
    const SampleLayout& sm = L.samples[b];
    // gen queries: gen keys (all, or the frames of the temporal window) + every valid ref run.
    // With a window, query tiles are cut per gen frame so that a tile shares one key set.
    const std::vector<RowRun> ref_runs = valid_runs(sm, 0, sm.R);
    auto gen_class = [&](int64_t row0, int64_t rows, int64_t key0, int64_t keys) {
      TileClass c{0, row0, rows, int32_t(s->spans.size()), 0, b, 0};
      s->spans.push_back({0, int32_t(key0), int32_t(keys), 0});
      for (const RowRun& r : ref_runs)
        s->spans.push_back({1, int32_t(sm.ref_off + r.r0), int32_t(r.r1 - r.r0), 0});
      c.span_cnt = int32_t(s->spans.size()) - c.span_off;
      classes.push_back(c);
    };
    if (sm.window < 0) {
      gen_class(sm.gen_off, sm.G, sm.gen_off, sm.G);
    } else {
      for (int32_t t = 0; t < sm.gen_frames; ++t) {
        const Run w = gen_window_frames(sm, t);
        gen_class(sm.gen_off + t * sm.Fg, sm.Fg, sm.gen_off + w.f0 * sm.Fg, (w.f1 - w.f0) * sm.Fg);
      }
    }
    if (L.gen_only) continue;
    // ref queries: per group, keys = valid runs of the group; query tiles per valid run
    for (int32_t g0 = 0; g0 < sm.ref_frames; g0 += sm.group) {
      const RowRun gr = group_rows(sm, g0);
      std::vector<RowRun> runs = valid_runs(sm, gr.r0, gr.r1);
      if (runs.empty()) continue;
      int32_t off = int32_t(s->spans.size());
      for (const RowRun& r : runs)
        s->spans.push_back({1, int32_t(sm.ref_off + r.r0), int32_t(r.r1 - r.r0), 0});
      for (const RowRun& r : runs)
        classes.push_back({1, sm.ref_off + r.r0, r.r1 - r.r0, off, int32_t(runs.size()), b, 0});
    }
  }
  CostedItems v;
  size_t n = 0;
  for (const TileClass& c : classes) n += size_t(L.heads) * size_t((c.rows + tile - 1) / tile);
  v.reserve(n);
  for (const TileClass& c : classes) emit_items(c, tile, L.heads, step, s->spans, &v);
  return v;
}

// First frame of the ref group holding sample-relative ref row r.
int32_t group_of_row(const SampleLayout& s, int64_t r) {
  if (!s.gbound.empty()) {
    const auto it = std::upper_bound(s.gbound.begin(), s.gbound.end(), r);
    return int32_t(it - s.gbound.begin() - 1) * s.group;
  }
  return int32_t(r / s.F) / s.group * s.group;
}

// Key-major items (dK/dV): key tiles, query spans per class.
CostedItems key_major_items(const Layout& L, int tile, int step, Schedule* s) {
  std::vector<TileClass> classes;
  CostedItems v;
  s->spans.clear();
  std::map<std::vector<int32_t>, int32_t> lists;  // span list (flattened) -> offset
  auto intern = [&](const std::vector<Span>& l) {
    std::vector<int32_t> key;
    for (const Span& x : l) key.insert(key.end(), {x.stream, x.start, x.len, x.keys});
    auto it = lists.find(key);
    if (it != lists.end()) return it->second;
    const int32_t off = int32_t(s->spans.size());
    s->spans.insert(s->spans.end(), l.begin(), l.end());
    lists.emplace(std::move(key), off);
    return off;
  };
  for (int32_t b = 0; b < L.batch; ++b) {
    const SampleLayout& sm = L.samples[b];
    // gen keys are seen by the gen queries of the sample only (those of the frames within the
    // temporal window, if any: the window is symmetric, so key frame t' is seen from the same
    // frames that t' would see)
    if (sm.window < 0) {
      int32_t gq = int32_t(s->spans.size());
      s->spans.push_back({0, int32_t(sm.gen_off), int32_t(sm.G), 0});
      classes.push_back({0, sm.gen_off, sm.G, gq, 1, b, 0});
    } else {
      for (int32_t t = 0; t < sm.gen_frames; ++t) {
        const Run w = gen_window_frames(sm, t);
        int32_t gq = int32_t(s->spans.size());
        s->spans.push_back({0, int32_t(sm.gen_off + w.f0 * sm.Fg), int32_t((w.f1 - w.f0) * sm.Fg), 0});
        classes.push_back({0, sm.gen_off + t * sm.Fg, sm.Fg, gq, 1, b, 0});
      }
    }
    // valid ref keys are seen by every gen query of the sample and by the valid ref queries of
    // their group. Tiles run across group boundaries inside each run of valid rows (a group's
    // last tile would otherwise be mostly empty and still stream every gen query); a tile's
    // span for one group's ref queries carries the range of the tile's keys in that group.
    for (const auto& run : sm.vruns) {
      for (int64_t a = run.first; a < run.second; a += tile) {
        const int64_t e = std::min<int64_t>(a + tile, run.second);
        std::vector<Span> l{{0, int32_t(sm.gen_off), int32_t(sm.G), 0}};
        if (!L.gen_only) {
          for (int32_t g0 = group_of_row(sm, a); g0 < sm.ref_frames; g0 += sm.group) {
            const RowRun gr = group_rows(sm, g0);
            if (gr.r0 >= e) break;
            const int64_t lo = std::max(a, gr.r0), hi = std::min(e, gr.r1);
            if (lo >= hi) continue;
            const int32_t keys = (lo == a && hi == e) ? 0 : int32_t(((hi - a) << 16) | (lo - a));
            for (const RowRun& q : valid_runs(sm, gr.r0, gr.r1))
              l.push_back({1, int32_t(sm.ref_off + q.r0), int32_t(q.r1 - q.r0), keys});
          }
        }
        const int32_t off = intern(l);
        int64_t step_rows = 0;
        for (const Span& x : l) step_rows += (x.len + step - 1) / step * step;
        for (int32_t h = 0; h < L.heads; ++h) {
          WorkItem w;
          w.stream = 1;
          w.head = h;
          w.start = int32_t(sm.ref_off + a);
          w.len = int32_t(e - a);
          w.span_off = off;
          w.span_cnt = int32_t(l.size());
          w.sample = b;
          w.slot = 0;
          v.push_back({int64_t(tile) * step_rows, w});
        }
      }
    }
  }
  for (const TileClass& c : classes) emit_items(c, tile, L.heads, step, s->spans, &v);
  return v;
}

// A schedule of whole items in launch order.
void finish_whole(CostedItems& v, const Layout& L, int step, bool heads_in_turn, Schedule* s) {
  order_items(v, L.heads, heads_in_turn, s);
  if (L.heads % kNumXcd == 0) align_phases(step, s);
}

// ---- splitting

// Times of a kernel in units of one 64-row step of a 256-row work item.
struct KernelCost {
  double step;     // one step
  double item;     // prologue and epilogue of a work item
  double piece;    // more of that for a piece, whose fp32 sums are written and read again
  double combine;  // the combine launch
};

// When a launch of these times (and how many items take each), longest first, would end on kNumCus
// compute units. Heads and tiles repeat a few times over, so whole groups of units take whole
// groups of items: the replay's cost goes with the kinds of items, not with their number (the whole
// plan of the 480p layer's 5 heads: 4.4 -> 0.48 ms on the host).
double makespan(std::vector<std::pair<double, int64_t>>& t) {
  std::sort(t.begin(), t.end(), std::greater<std::pair<double, int64_t>>());
  std::map<double, int64_t> free_at{{0.0, kNumCus}};  // compute units by the time they are free
  double end = 0;
  for (const auto& [x, count] : t)
    for (int64_t left = count; left > 0;) {
      const auto first = free_at.begin();
      const double done = first->first + x;
      const int64_t n = std::min(left, first->second);
      left -= n;
      if ((first->second -= n) == 0) free_at.erase(first);
      free_at[done] += n;
      end = std::max(end, done);
    }
  return end;
}

int32_t span_steps(const Span& x) { return (x.len + kStep - 1) / kStep; }

constexpr int kSplitRounds = 8;

// An item of a launch: its steps, its kernel's times and the bytes of a piece's partial results.
struct Timed {
  int32_t steps;
  const KernelCost* c;
  int64_t bytes;
  double time() const { return steps * c->step + c->item; }
};

// Microseconds that writing and reading these partial results adds to a launch: little while the
// caches hold them (12 heads of 220 + 330 tokens, 49 MB: the split backward 60 -> 50 us), up to
// 1 TB/s beyond (5 heads of 3,060 + 2,142 tokens, 80 MB: 40 us over the end replayed without them).
double partials_us(int64_t bytes) {
  constexpr int64_t kCached = int64_t(64) << 20;
  return double(bytes) / 10e6 + double(std::max<int64_t>(0, bytes - kCached)) / 1e6;
}

// Pieces per item (same order as `v`, which is longest first) that end the launch earliest, or
// all ones; *end is that time. Tried: every item longer than a part of the longest cut to such
// parts, and the same for only those items of the long ones that a last, partial round of the
// compute units would hold. Not for launches of over kSplitRounds rounds: there the order that keeps
// items of a head in step on an XCD is worth more than the last round. unit_us: one unit of the
// times in microseconds. A launch that ends before `least` stays whole.
std::vector<int32_t> choose_split(const std::vector<Timed>& v, int64_t max_bytes, double unit_us, double least, bool exact,
                                  double* end) {
  const size_t n = v.size();
  std::vector<int32_t> best(n, 1);
  *end = 0;
  if (n == 0) return best;
  if (n > size_t(kSplitRounds * kNumCus)) {
    double total = 0;
    for (const Timed& x : v) total += x.time();
    *end = total / kNumCus + 0.5 * v[0].time();
    return best;
  }
  const double longest = v[0].steps * v[0].c->step;
  size_t n_long = 0;
  while (n_long < n && 2 * v[n_long].time() >= v[0].time()) ++n_long;
  const size_t rounds = n_long / kNumCus * kNumCus;
  std::vector<size_t> at;  // where runs of like items begin, and the end; also the first of the last round
  for (size_t i = 0; i < n; ++i)
    if (i == 0 || i == rounds || v[i].steps != v[i - 1].steps || v[i].c != v[i - 1].c) at.push_back(i);
  at.push_back(n);
  const size_t m = at.size() - 1;
  std::vector<int32_t> chosen(m, 1), k(m, 1), last;
  std::vector<std::pair<double, int64_t>> t;
  // the launch's end, or any value over `bound` where it ends later than that
  auto eval = [&](const std::vector<int32_t>& parts, int64_t bytes, double bound) {
    t.clear();
    double combine = 0, total = 0, most = 0;
    for (size_t r = 0; r < m; ++r) {
      const Timed& x = v[at[r]];
      const KernelCost& c = *x.c;
      if (parts[r] > 1) combine = std::max(combine, c.combine);
      const double time = double(x.steps) / parts[r] * c.step + c.item + (parts[r] > 1 ? c.piece : 0);
      const int64_t count = int64_t(at[r + 1] - at[r]) * parts[r];
      t.push_back({time, count});
      most = std::max(most, time);
      total += time * count;
    }
    const double more = combine + partials_us(bytes) / unit_us, least_end = std::max(most, total / kNumCus);
    return least_end + more > bound ? least_end + more : makespan(t) + more;
  };
  *end = eval(chosen, 0, HUGE_VAL);
  const double whole = *end;
  if (whole < least) return best;
  // lengths of the pieces: whole parts of the longest item's; with `exact` also those at which the number
  // of another long item's pieces changes, up to four (kinds of items then divide evenly)
  std::vector<double> lengths;
  for (int32_t parts = 2; parts <= 24; ++parts) lengths.push_back(longest / parts);
  for (size_t r = 0; exact && r < m; ++r) {
    const double x = v[at[r]].steps * v[at[r]].c->step;
    for (int32_t parts = 1; parts <= 4 && 2 * x >= longest; ++parts)
      if (x < parts * longest && 4 * x > parts * longest) lengths.push_back(x / parts);
  }
  std::sort(lengths.begin(), lengths.end(), std::greater<double>());
  for (double length : lengths) {
    for (int tail = 0; tail < (rounds > 0 ? 2 : 1); ++tail) {
      int64_t bytes = 0;
      for (size_t r = 0; r < m; ++r) {
        const Timed& x = v[at[r]];
        const double piece = std::max(2.0 * x.c->step, length);  // two steps at least
        k[r] = at[r] < (tail ? rounds : 0) ? 1 : std::max<int32_t>(1, int32_t(std::ceil(x.steps * x.c->step / piece - 1e-9)));
        if (k[r] > 1) bytes += k[r] * x.bytes * int64_t(at[r + 1] - at[r]);
      }
      if (bytes == 0 || bytes > max_bytes || k == last) continue;  // pieces no longer get shorter
      last = k;
      const double bound = std::min((exact ? 0.98 : 1.0) * *end, 0.97 * whole);
      const double e = eval(k, bytes, bound);
      if (e < bound) {
        *end = e;
        chosen = k;
      }
    }
  }
  for (size_t r = 0; r < m; ++r) std::fill(best.begin() + at[r], best.begin() + at[r + 1], chosen[r]);
  return best;
}

// Replaces the items of v (longest first, with their spans in s) by their pieces, into s: parts[i]
// pieces of like numbers of steps each, at most as many as the item has steps.
void split_items(const CostedItems& v, const std::vector<int32_t>& parts, Schedule* s) {
  std::vector<Span> spans;
  std::map<std::pair<int32_t, std::pair<int32_t, int32_t>>, std::pair<int32_t, int32_t>> made;
  std::vector<std::pair<int32_t, WorkItem>> out;
  // steps [s0, s1) of a span list as a list of its own: its offset and length
  auto cut = [&](const WorkItem& w, int32_t s0, int32_t s1) {
    const auto key = std::make_pair(w.span_off, std::make_pair(s0, s1));
    const auto it = made.find(key);
    if (it != made.end()) return it->second;
    const int32_t off = int32_t(spans.size());
    int32_t at = 0;
    for (int32_t i = 0; i < w.span_cnt && at < s1; ++i) {
      const Span& x = s->spans[size_t(w.span_off) + i];
      const int32_t m = span_steps(x), a = std::max(s0, at) - at, b = std::min(s1, at + m) - at;
      if (a < b) spans.push_back({x.stream, x.start + a * kStep, std::min(x.len, b * kStep) - a * kStep, x.keys});
      at += m;
    }
    return made[key] = {off, int32_t(spans.size()) - off};
  };
  for (size_t i = 0; i < v.size(); ++i) {
    const WorkItem& w = v[i].second;
    int32_t steps = 0;
    for (int32_t j = 0; j < w.span_cnt; ++j) steps += span_steps(s->spans[size_t(w.span_off) + j]);
    const int32_t k = parts[i];
    if (k > 1) s->combine.push_back({w.stream, w.head, w.start, w.len, s->slots, k, {0, 0}});
    int32_t from = 0;
    for (int32_t j = 1; j <= k; ++j) {
      const int32_t to = int32_t(int64_t(steps) * j / k);
      WorkItem x = w;
      const auto c = cut(w, from, to);
      x.span_off = c.first;
      x.span_cnt = c.second;
      x.slot = k > 1 ? ++s->slots : 0;
      out.push_back({to - from, x});
      from = to;
    }
  }
  std::stable_sort(out.begin(), out.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
  s->items.clear();
  for (auto& e : out) s->items.push_back(e.second);
  s->real_items = int64_t(s->items.size());
  s->spans.swap(spans);
}

// Leaves of the launch of all rows what the call of the gen queries alone needs: query items and
// pieces of the gen rows; of the key items and pieces of split_items (key_major) the gen queries'
// spans, which come first in every list. The gen rows' sums then run in one order whether or not the
// reference queries are computed. Slots are numbered anew, and an item left with one piece is whole:
// what is dropped would only have added zeros (a reference query whose output has no gradient).
// `heads` as in deal_items, or 1 where items are not dealt to the XCDs.
void keep_gen_queries(bool key_major, int32_t heads, Schedule* s) {
  std::vector<WorkItem> items;
  std::vector<Span> spans;
  std::map<std::pair<int32_t, int32_t>, int32_t> made;  // (span list's offset, spans kept) -> new offset
  std::vector<int32_t> slot(size_t(s->slots) + 1, 0);   // old slot -> 1 if kept, then the new slot
  items.reserve(s->items.size());
  int32_t last_off = -1, last_cnt = -1, last_new = 0;  // items of one list mostly follow one another
  for (WorkItem w : s->items) {
    if (w.stream < 0) continue;
    const Span* l = &s->spans[size_t(w.span_off)];
    if (key_major) {
      int32_t n = 0;
      while (n < w.span_cnt && l[n].stream == 0) ++n;
      w.span_cnt = n;
    }
    if (key_major ? w.span_cnt == 0 : w.stream != 0) continue;
    if (w.span_off != last_off || w.span_cnt != last_cnt) {
      const auto at = made.emplace(std::make_pair(w.span_off, w.span_cnt), int32_t(spans.size()));
      if (at.second) spans.insert(spans.end(), l, l + w.span_cnt);
      last_off = w.span_off;
      last_cnt = w.span_cnt;
      last_new = at.first->second;
    }
    w.span_off = last_new;
    if (w.slot) slot[size_t(w.slot)] = 1;
    items.push_back(w);
  }
  std::vector<CombineItem> combine;
  s->slots = 0;
  for (CombineItem c : s->combine) {
    const auto first = slot.begin() + c.slot0 + 1, last = first + c.n;
    c.slot0 = s->slots;
    c.n = int32_t(std::count(first, last, 1));
    for (auto x = first; x != last; ++x)
      if (*x) *x = c.n > 1 ? ++s->slots : 0;
    if (c.n > 1) combine.push_back(c);
  }
  for (WorkItem& w : items) w.slot = slot[size_t(w.slot)];
  s->spans.swap(spans);
  s->combine.swap(combine);
  deal_items(items, heads, s);
}

// Sorts v longest first and returns the items' steps.
std::vector<int32_t> sort_steps(CostedItems& v, const Schedule& s) {
  longest_first(v);
  std::map<std::pair<int32_t, int32_t>, int32_t> known;
  std::vector<int32_t> steps;
  steps.reserve(v.size());
  auto it = known.end();
  for (const auto& e : v) {  // items of one span list mostly follow one another
    const auto key = std::make_pair(e.second.span_off, e.second.span_cnt);
    if (it == known.end() || it->first != key) it = known.find(key);
    if (it == known.end()) {
      int32_t n = 0;
      for (int32_t i = 0; i < key.second; ++i) n += span_steps(s.spans[size_t(key.first) + i]);
      it = known.emplace(key, n).first;
    }
    steps.push_back(it->second);
  }
  return steps;
}

// The forward's partial results take no more than kFwdPartialBytes. kTableBytes is more than the tables
// of a split launch (at most kSplitRounds rounds of items and their pieces) take, but for calls whose
// span lists hold thousands of short runs.
constexpr int64_t kTableBytes = int64_t(4) << 20;
constexpr int64_t kFwdPartialBytes = int64_t(SRA_NOALLOC_WORKSPACE_MAX) - kTableBytes;

constexpr double kFwdUnitUs = 1.5;  // a 64-key step of 256 rows at d = 128 (1.1 at d = 64)

// Launches that end before this take about as long as the host's part of a call, which a split makes a
// launch longer. d = 64, items of up to 16 steps: calls in a row 27.4-29.0 us whole, 29.6-32.0 split
// (a call waited for 52-55 and 47-52); of 17 to 19 steps 27.5-32.7 and 19.5-27.5. d = 128, 9 and 10
// steps: 21.6-31.2 whole, 19.9-31.3 split. Steps of items of up to 128 rows, one wave per SIMD, take
// 0.7 of the time (128 and 192 rows: 0.76 and 1.09 us at d = 128, 0.66 and 0.97 at d = 64): of 9 and
// 10 steps at d = 128 23.7 and 28.7 whole, 26.2 and 30.8 split.
constexpr double kFwdLeast[2] = {19.5, 11.5};  // d = 64, 128
constexpr double kFwdHalfStep = 0.7;

// A schedule of the call of all rows with whole 256-row items.
void whole_forward_schedule(const Layout& L, Schedule* out) {
  CostedItems v = query_major_items(L, kFwdQueryTile, kFwdKeyStep, out);
  out->tile = kFwdQueryTile;
  out->mfma32 = true;
  finish_whole(v, L, kFwdKeyStep, false, out);
}

// The forward's launch of all rows: rows per item and splits by the replayed end. A step of the large
// tile holds 1.5 (d = 128) or 2 (d = 64) times the rows and takes 1.36 or 1.78 times as long (480p, 40
// heads: 25.5 -> 23.7 ms; 480p, d = 64, 16 heads: 8.11 -> 7.18 ms). max_bytes: of partial results.
// Returns whether items are split.
// 256-row items run on 32x32x16 MFMAs (mfma32) but for d = 128 where the launch fills the chip for long
// enough that the board's power limit sets in: more items than compute units, of 20 steps or more,
// 110 us of steps each. There 16x16x32 MFMAs are the faster (840 items, 286 us: 4 %; 743, 2.18 ms: 3.5 %;
// 352, 181 us: 2.5 %), elsewhere 32x32x16 ones (148 items, 394 us: 10 %; 456, 109 us: 8 %; 1,840 of 13
// steps, 192 us: 6 %). At d = 64 they are at every size (2.44 ms: 5 %).
bool best_forward_schedule(const Layout& L, int64_t max_bytes, Schedule* out) {
  double least = kFwdLeast[L.head_dim == 128];
  double best = 0, total = 0;
  CostedItems v;
  std::vector<int32_t> parts;
  for (int tile : {kFwdQueryTile, fwd_large_tile(L.head_dim)}) {
    const bool large = tile != kFwdQueryTile;
    const KernelCost c{!large ? 1.0 : L.head_dim == 128 ? 1.36 : 1.78, 3.0, large ? 3.0 : 2.0, L.head_dim == 128 ? 4.0 : 7.0};
    Schedule s;
    CostedItems items = query_major_items(L, tile, kFwdKeyStep, &s);
    const std::vector<int32_t> steps = sort_steps(items, s);
    std::vector<Timed> timed;
    timed.reserve(steps.size());
    for (int32_t n : steps) timed.push_back({n, &c, slot_bytes(tile, L.head_dim, 1, 2)});
    if (!large) {  // the rows of the items that decide when the launch ends
      int32_t rows = 0;
      for (size_t i = 0; i < items.size() && 2 * steps[i] >= steps[0]; ++i) rows = std::max(rows, items[i].second.len);
      if (rows <= kFwdQueryTile / 2) least /= kFwdHalfStep;
    }
    double end;
    std::vector<int32_t> k = choose_split(timed, max_bytes, kFwdUnitUs, least, false, &end);
    if (large && !(end < 0.99 * best)) continue;
    best = end;
    total = std::accumulate(steps.begin(), steps.end(), 0.0);
    s.tile = tile;
    v.swap(items);
    parts.swap(k);
    *out = std::move(s);
    if (best < least && std::all_of(parts.begin(), parts.end(), [](int32_t k) { return k == 1; })) break;
  }
  const bool split = std::any_of(parts.begin(), parts.end(), [](int32_t k) { return k > 1; });
  const double n = std::accumulate(parts.begin(), parts.end(), 0.0);
  out->mfma32 = out->tile == kFwdQueryTile &&
                (L.head_dim == 64 || n <= kNumCus || total < 20 * n || total * kFwdUnitUs < 110.0 * kNumCus);
  if (split) split_items(v, parts, out);
  else finish_whole(v, L, kFwdKeyStep, false, out);
  return split;
}

// The forward's launch. `fixed`: the rest of its workspace. Where that leaves room in the static scratch
// of the allocation-free forward, the tables and partial results stay within it wherever those of
// whole 256-row items do, so that it takes the same calls and runs the same launch.
void launch_forward_schedule(const Layout& L, int64_t fixed, Schedule* out) {
  Layout all = L;
  all.gen_only = false;
  const int64_t room = int64_t(SRA_NOALLOC_WORKSPACE_MAX) - fixed;  // <= 0: it rejects the call anyway
  auto need = [&](const Schedule& s) {
    return int64_t(s.items.size() * sizeof(WorkItem) + s.spans.size() * sizeof(Span) +
                   s.combine.size() * sizeof(CombineItem)) + s.slots * slot_bytes(s.tile, L.head_dim, 1, 2);
  };
  int64_t bytes = room <= 0 ? kFwdPartialBytes : std::max<int64_t>(0, std::min(kFwdPartialBytes, room - kTableBytes));
  bool split = best_forward_schedule(all, bytes, out);
  for (bool last : {false, true}) {  // larger tables than reckoned: as much less for the partial results, or none
    if (room <= 0 || need(*out) <= room || !split) break;
    bytes = last ? 0 : std::max<int64_t>(0, bytes - (need(*out) - room));
    *out = Schedule();
    split = best_forward_schedule(all, bytes, out);
  }
  if (room > 0 && need(*out) > room) {  // phases of the larger tile may copy long span lists more often
    Schedule s;
    whole_forward_schedule(all, &s);
    if (need(s) <= room) *out = std::move(s);
  }
  if (L.gen_only) keep_gen_queries(false, split ? 1 : L.heads, out);
}

// The backward's launches. Times in units of 0.75 us: a dQ step takes 2.25 us and a dK/dV step 3.0
// at d = 128 (1.4 and 1.85 at d = 64), a launch and its first tile about 6. Up to kSplitRounds rounds
// of items run as one launch, split where that ends earlier; longer launches run kind by kind,
// each in its own order.
constexpr int64_t kBwdPartialBytes = int64_t(256) << 20;
constexpr double kBwdUnitUs = 0.75;
const KernelCost kDkvCosts[2] = {{2.4, 8.0, 8.0, 8.0}, {4.0, 8.0, 8.0, 8.0}};  // d = 64, 128
const KernelCost kDqCosts[2] = {{1.8, 8.0, 5.0, 8.0}, {3.0, 8.0, 5.0, 8.0}};

void launch_backward_schedules(const Layout& L, Plan* plan) {
  // Whether and how items are split is settled for the call of all rows, so that the gradients of
  // the gen rows and of the keys do not depend on whether the ref queries are computed.
  Layout full = L;
  full.gen_only = false;
  Schedule dq, dkv;
  CostedItems vq = query_major_items(full, kDqQueryTile, kStep, &dq);
  CostedItems vk = key_major_items(full, kDkvKeyTile, kStep, &dkv);
  dq.tile = kDqQueryTile;
  dkv.tile = kDkvKeyTile;
  if (vq.size() + vk.size() > size_t(kSplitRounds * kNumCus)) {
    finish_whole(vq, L, kStep, false, &dq);
    if (L.gen_only) {
      keep_gen_queries(false, L.heads, &dq);
      dkv = Schedule();
      vk = key_major_items(L, kDkvKeyTile, kStep, &dkv);
      dkv.tile = kDkvKeyTile;
    }
    finish_whole(vk, L, kStep, true, &dkv);
    plan->dq = std::move(dq);
    plan->dkv = std::move(dkv);
    return;
  }
  // entry i < vk.size(): key item i, else query item i - vk.size()
  const KernelCost &dkv_cost = kDkvCosts[L.head_dim == 128], &dq_cost = kDqCosts[L.head_dim == 128];
  const std::vector<int32_t> sk = sort_steps(vk, dkv), sq = sort_steps(vq, dq);
  std::vector<Timed> timed, sorted;
  timed.reserve(sk.size() + sq.size());
  sorted.reserve(sk.size() + sq.size());
  for (int32_t n : sk) timed.push_back({n, &dkv_cost, slot_bytes(kDkvKeyTile, L.head_dim, 2, 0)});
  for (int32_t n : sq) timed.push_back({n, &dq_cost, slot_bytes(kDqQueryTile, L.head_dim, 1, 0)});
  std::vector<int32_t> order(timed.size());
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return timed[a].time() > timed[b].time(); });
  for (int32_t i : order) sorted.push_back(timed[i]);
  double end;
  const std::vector<int32_t> k = choose_split(sorted, kBwdPartialBytes, kBwdUnitUs, 0, true, &end);
  std::vector<int32_t> pk(vk.size()), pq(vq.size());
  for (size_t i = 0; i < order.size(); ++i) {
    if (size_t(order[i]) < vk.size()) pk[order[i]] = k[i];
    else pq[order[i] - vk.size()] = k[i];
  }
  split_items(vk, pk, &dkv);
  split_items(vq, pq, &dq);
  if (L.gen_only) {
    keep_gen_queries(true, 1, &dkv);
    keep_gen_queries(false, 1, &dq);
  }
  Schedule& g = plan->grad;
  std::vector<std::pair<double, WorkItem>> all;
  auto add = [&](const Schedule& s, const KernelCost& c, int32_t mark) {
    const int32_t base = int32_t(g.spans.size());
    g.spans.insert(g.spans.end(), s.spans.begin(), s.spans.end());
    for (WorkItem w : s.items) {
      int32_t n = 0;
      for (int32_t i = 0; i < w.span_cnt; ++i) n += span_steps(s.spans[size_t(w.span_off) + i]);
      w.span_off += base;
      w.stream |= mark;
      all.push_back({n * c.step + c.item, w});
    }
    g.combine.insert(g.combine.end(), s.combine.begin(), s.combine.end());
  };
  add(dkv, dkv_cost, 0);
  add(dq, dq_cost, 2);
  std::stable_sort(all.begin(), all.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
  for (auto& e : all) g.items.push_back(e.second);
  g.real_items = int64_t(g.items.size());
  plan->grad_joint = true;
  plan->grad_kv_combine = int32_t(dkv.combine.size());
  for (auto [from, to] : {std::make_pair(&dq, &plan->dq), std::make_pair(&dkv, &plan->dkv)}) {
    to->tile = from->tile;
    to->slots = from->slots;
  }
}

}  // namespace

bool needs_compaction(const Layout& L) {
  for (const SampleLayout& s : L.samples) {
    int64_t groups = 0;
    for (int32_t g0 = 0; g0 < s.ref_frames; g0 += s.group) {
      const RowRun gr = group_rows(s, g0);
      if (!valid_runs(s, gr.r0, gr.r1).empty()) ++groups;
    }
    if (int64_t(s.vruns.size()) > groups) return true;
  }
  return false;
}

void compact_layout(const Layout& L, Layout* C, std::vector<int32_t>* gather, std::vector<int32_t>* scatter) {
  *C = L;
  C->sum_ref = 0;
  gather->clear();
  scatter->assign(size_t(L.sum_ref), -1);
  for (size_t b = 0; b < L.samples.size(); ++b) {
    const SampleLayout& s = L.samples[b];
    SampleLayout& c = C->samples[b];
    c.ref_off = C->sum_ref;
    c.gbound.assign(1, 0);
    int64_t n = 0;
    for (int32_t g0 = 0; g0 < s.ref_frames; g0 += s.group) {
      const RowRun gr = group_rows(s, g0);
      for (const RowRun& r : valid_runs(s, gr.r0, gr.r1))
        for (int64_t row = r.r0; row < r.r1; ++row, ++n) {
          (*scatter)[size_t(s.ref_off + row)] = int32_t(c.ref_off + n);
          gather->push_back(int32_t(s.ref_off + row));
        }
      c.gbound.push_back(n);
    }
    c.R = n;
    c.vruns.clear();
    if (n > 0) c.vruns.push_back({0, n});
    C->sum_ref += n;
  }
}

void build_plan(const Layout& L_in, Plan* plan, bool whole) {
  plan->layout = L_in;
  plan->compacted = needs_compaction(L_in);
  plan->ref_gather.clear();
  plan->ref_scatter.clear();
  if (plan->compacted)
    compact_layout(L_in, &plan->exec, &plan->ref_gather, &plan->ref_scatter);
  else
    plan->exec = L_in;
  const Layout& L = plan->exec;
  plan->fill.clear();
  for (const SampleLayout& sm : L.samples) {  // the gaps between valid ref runs
    int64_t r = 0;
    for (const auto& v : sm.vruns) {
      if (v.first > r) plan->fill.push_back({1, int32_t(sm.ref_off + r), int32_t(v.first - r), 0});
      r = v.second;
    }
    if (r < sm.R) plan->fill.push_back({1, int32_t(sm.ref_off + r), int32_t(sm.R - r), 0});
  }
  plan->fwd = plan->dq = plan->dkv = Schedule();
  if (whole) {
    whole_forward_schedule(L, &plan->fwd);
  } else {
    int64_t fixed = int64_t(plan->fill.size() * sizeof(FillRange)) + 16 * 256;  // and every part's alignment
    if (plan->compacted) fixed += L.sum_ref * (L.heads * (8 * int64_t(L.head_dim) + 4) + 4) + L_in.sum_ref * 4;
    launch_forward_schedule(L, fixed, &plan->fwd);
  }
  plan->grad_joint = false;
  plan->grad = Schedule();
  if (whole) {
    CostedItems vq = query_major_items(L, kDqQueryTile, kDqKeyStep, &plan->dq);
    finish_whole(vq, L, kDqKeyStep, false, &plan->dq);
    CostedItems vk = key_major_items(L, kDkvKeyTile, kDkvQueryStep, &plan->dkv);
    finish_whole(vk, L, kDkvQueryStep, true, &plan->dkv);
  } else {
    launch_backward_schedules(L, plan);
  }
}

int64_t covered_pairs(const Schedule& s, bool /*key_major*/) {
  int64_t n = 0;
  for (const WorkItem& w : s.items) {
    if (w.stream < 0 || w.head != 0) continue;
    for (int32_t i = 0; i < w.span_cnt; ++i) {
      const Span& x = s.spans[w.span_off + i];
      const int64_t keys = x.keys ? (x.keys >> 16) - (x.keys & 0xffff) : w.len;
      n += keys * x.len;
    }
  }
  return n;
}

std::string layout_key(const Layout& L) {
  std::string k;
  auto put = [&k](int64_t v) { k.append(reinterpret_cast<const char*>(&v), sizeof v); };
  put(L.batch); put(L.heads); put(L.head_dim); put(L.gen_only ? 1 : 0);
  for (const SampleLayout& s : L.samples) {
    put(s.G); put(s.R); put(s.F); put(s.Fg); put(s.ref_frames); put(s.group); put(s.window);
    put(int64_t(s.vruns.size()));
    for (const auto& r : s.vruns) { put(r.first); put(r.second); }
  }
  return k;
}

}  // namespace sra
