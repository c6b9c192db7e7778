// Host side of the library: block planner, descriptor validation, work-queue scheduler.
// Integer work only; the only HIP calls are the workspace upload in fcp_queue_build.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <mutex>
#include <numeric>
#include <queue>
#include <unordered_map>
#include <utility>
#include <vector>

#include "fcp_internal.h"
#include "fcp_probe.h"

namespace fcp {

static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
}

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

int validate_problem(const fcp_problem* p) {
  if (!p) { set_error("problem descriptor is NULL"); return FCP_ERR_INVALID_ARG; }
  if (p->n_q_heads <= 0 || p->n_kv_heads <= 0 || p->block_size <= 0) {
    set_error("heads and block_size must be positive"); return FCP_ERR_INVALID_ARG;
  }
  if (p->head_dim != 64 && p->head_dim != 128) {
    set_error("head_dim %d unsupported (64 or 128)", p->head_dim); return FCP_ERR_UNSUPPORTED;
  }
  if (p->n_q_heads % p->n_kv_heads != 0) {
    set_error("n_q_heads %d is not a multiple of n_kv_heads %d", p->n_q_heads, p->n_kv_heads);
    return FCP_ERR_UNSUPPORTED;
  }
  if (p->n_kv_blocks < 0 || p->n_q_blocks < 0 || p->n_pairs < 0 || p->n_slots < 0 || p->n_slot_rows < 0) {
    set_error("negative table count"); return FCP_ERR_INVALID_ARG;
  }
  if ((p->n_kv_blocks && !p->kv_blocks) || (p->n_q_blocks && !p->q_blocks) || (p->n_pairs && !p->pairs) ||
      (p->n_slots && !p->slots)) {
    set_error("NULL table with a non-zero count"); return FCP_ERR_INVALID_ARG;
  }
  if (!(p->softmax_scale >= 0.0f)) { set_error("softmax_scale must be >= 0 (0 = 1/sqrt(d))"); return FCP_ERR_INVALID_ARG; }
  if (p->n_segments < 0 || (p->n_segments && !p->segments)) { set_error("segments: negative count or NULL table"); return FCP_ERR_INVALID_ARG; }
  int64_t tok = 0;
  for (int i = 0; i < p->n_kv_blocks; i++) {
    const fcp_block& b = p->kv_blocks[i];
    if (b.tok_len <= 0 || b.tok_len > p->block_size || b.tok_start != tok) {
      set_error("kv_blocks[%d]: tok_len/tok_start inconsistent (blocks must be packed in order)", i);
      return FCP_ERR_INVALID_ARG;
    }
    tok += b.tok_len;
    if (tok > INT32_MAX) { set_error("more than 2^31-1 KV tokens"); return FCP_ERR_UNSUPPORTED; }
  }
  tok = 0;
  for (int i = 0; i < p->n_q_blocks; i++) {
    const fcp_block& b = p->q_blocks[i];
    if (b.tok_len <= 0 || b.tok_len > p->block_size || b.tok_start != tok) {
      set_error("q_blocks[%d]: tok_len/tok_start inconsistent (blocks must be packed in order)", i);
      return FCP_ERR_INVALID_ARG;
    }
    tok += b.tok_len;
  }
  // members of packed blocks: by (kv_blk, tok_off), tiling their block exactly
  std::vector<char> segmented;
  std::vector<int32_t> first_seg;              // of each packed KV block
  if (p->n_segments) {
    segmented.assign(p->n_kv_blocks, 0);
    first_seg.assign(p->n_kv_blocks, 0);
    int32_t blk = -1, covered = 0;
    for (int i = 0; i <= p->n_segments; i++) {
      if (i == p->n_segments || p->segments[i].kv_blk != blk) {
        if (blk >= 0 && covered != p->kv_blocks[blk].tok_len) {
          set_error("segments: the members of kv block %d do not cover it", blk); return FCP_ERR_INVALID_ARG;
        }
        if (i == p->n_segments) break;
        const int32_t nb = p->segments[i].kv_blk;
        if (nb <= blk || nb >= p->n_kv_blocks) { set_error("segments[%d]: kv_blk out of range or not ascending", i); return FCP_ERR_INVALID_ARG; }
        if (p->kv_blocks[nb].tok_len > kMaxPackedBlock) { set_error("segments[%d]: a packed block holds at most %d tokens", i, kMaxPackedBlock); return FCP_ERR_UNSUPPORTED; }
        blk = nb; covered = 0; segmented[nb] = 1; first_seg[nb] = i;
      }
      const fcp_segment& sg = p->segments[i];
      if (sg.tok_off != covered || sg.tok_len <= 0 || (int64_t)sg.tok_off + sg.tok_len > p->kv_blocks[blk].tok_len) {
        set_error("segments[%d]: members must follow each other inside their block", i); return FCP_ERR_INVALID_ARG;
      }
      covered += sg.tok_len;
    }
  }
  // the rows of a packed query block are cut up once: its PACKED pairs must join KV blocks with the same members
  auto same_members = [&](int32_t a, int32_t b) {
    for (int32_t i = first_seg[a], j = first_seg[b]; a != b; i++, j++) {
      const bool in_a = i < p->n_segments && p->segments[i].kv_blk == a, in_b = j < p->n_segments && p->segments[j].kv_blk == b;
      if (!in_a || !in_b) return in_a == in_b;
      if (p->segments[i].tok_len != p->segments[j].tok_len) return false;
    }
    return true;
  };
  int prev_q = -1, packed_kv = -1;
  int64_t pair_cursor = 0;
  for (int s = 0; s < p->n_slots; s++) {
    const fcp_slot& sl = p->slots[s];
    if (sl.q_blk < 0 || sl.q_blk >= p->n_q_blocks || sl.q_blk < prev_q) {
      set_error("slots[%d]: q_blk out of range or not ascending", s); return FCP_ERR_INVALID_ARG;
    }
    if (sl.q_blk != prev_q) packed_kv = -1;
    prev_q = sl.q_blk;
    if (sl.pair_begin != pair_cursor || sl.n_pairs < 0 || pair_cursor + sl.n_pairs > p->n_pairs) {
      set_error("slots[%d]: pair range must continue where the previous slot ended", s);
      return FCP_ERR_INVALID_ARG;
    }
    pair_cursor += sl.n_pairs;
    const int qlen = p->q_blocks[sl.q_blk].tok_len;
    if (sl.row_start < 0 || (int64_t)sl.row_start + qlen > p->n_slot_rows) {
      set_error("slots[%d]: rows outside the partial buffers", s); return FCP_ERR_INVALID_ARG;
    }
    for (int64_t i = sl.pair_begin; i < sl.pair_begin + sl.n_pairs; i++) {
      const fcp_pair& pr = p->pairs[i];
      if (pr.q_blk != sl.q_blk || pr.slot != s || pr.kv_blk < 0 || pr.kv_blk >= p->n_kv_blocks ||
          pr.kind < FCP_KIND_FULL || pr.kind > FCP_KIND_PACKED_DIAG) {
        set_error("pairs[%lld]: inconsistent with slot %d", (long long)i, s); return FCP_ERR_INVALID_ARG;
      }
      if (pr.kind != FCP_KIND_FULL) {
        const fcp_block& qb = p->q_blocks[pr.q_blk];
        const fcp_block& kb = p->kv_blocks[pr.kv_blk];
        if (qb.seq != kb.seq || qb.idx != kb.idx || qb.tok_len != kb.tok_len) {
          set_error("pairs[%lld]: a DIAG or PACKED pair must join a block with itself", (long long)i);
          return FCP_ERR_INVALID_ARG;
        }
      }
      const bool seg = !segmented.empty() && segmented[pr.kv_blk];
      if (seg != ((pr.kind & 2) != 0)) {
        set_error("pairs[%lld]: a PACKED kind needs a KV block with members, the other kinds one without", (long long)i);
        return FCP_ERR_INVALID_ARG;
      }
      if ((pr.kind & 2) && sl.n_pairs != 1) {
        set_error("pairs[%lld]: a packed query block has one pair", (long long)i); return FCP_ERR_INVALID_ARG;
      }
      if (pr.kind & 2) {
        if (packed_kv >= 0 && !same_members(packed_kv, pr.kv_blk)) {
          set_error("pairs[%lld]: the PACKED pairs of a query block must join KV blocks with the same members", (long long)i);
          return FCP_ERR_INVALID_ARG;
        }
        packed_kv = pr.kv_blk;
      }
    }
  }
  if (pair_cursor != p->n_pairs) { set_error("slots do not cover all pairs"); return FCP_ERR_INVALID_ARG; }
  return FCP_OK;
}

namespace {

// Rows of a block that the kernels treat as one segment: all of a plain block, or whole members of a packed one
// (segments seg_begin .. of the problem; more than one: joined).
struct Run { int32_t off, len, seq, seg_begin, n_segs; };
struct Runs { std::vector<Run> run; std::vector<int32_t> begin; };   // of KV block b: begin[b] .. begin[b + 1]

// Rows of a query-stationary item: one row tile of two heads when the group size is even, else two row tiles of one head.
int item_rows(const fcp_problem* p) { return kFwdTileM * ((p->n_q_heads / p->n_kv_heads) % 2 == 0 ? 1 : 2); }

Runs make_runs(const fcp_problem* p) {
  Runs r;
  r.run.reserve(p->n_kv_blocks);
  const int most = item_rows(p);
  for (int b = 0, i = 0; b < p->n_kv_blocks; b++) {
    r.begin.push_back((int32_t)r.run.size());
    if (i == p->n_segments || p->segments[i].kv_blk != b) r.run.push_back({0, p->kv_blocks[b].tok_len, p->kv_blocks[b].seq, i, 0});
    for (; i < p->n_segments && p->segments[i].kv_blk == b; i++) {
      const fcp_segment& sg = p->segments[i];
      if ((int32_t)r.run.size() > r.begin[b] && r.run.back().len + sg.tok_len <= most) {
        r.run.back().len += sg.tok_len;
        r.run.back().n_segs++;
      } else {
        r.run.push_back({sg.tok_off, sg.tok_len, sg.seq, i, 1});
      }
    }
  }
  r.begin.push_back((int32_t)r.run.size());
  return r;
}

// f(query block, its slots s0 .. s1, its runs, n_runs, packed): the runs of its PACKED pairs' KV blocks (which all have the
// same members), or one run of all its rows.
template <class F>
void for_q_blocks(const fcp_problem* p, const Runs& runs, F f) {
  for (int b = 0, s = 0; b < p->n_q_blocks; b++) {
    const int s0 = s;
    int kb = -1;
    for (; s < p->n_slots && p->slots[s].q_blk == b; s++)
      if (p->slots[s].n_pairs == 1 && (p->pairs[p->slots[s].pair_begin].kind & 2)) kb = p->pairs[p->slots[s].pair_begin].kv_blk;
    const Run whole = {0, p->q_blocks[b].tok_len, p->q_blocks[b].seq, 0, 0};
    if (kb < 0) f(b, s0, s, &whole, 1, false);
    else f(b, s0, s, &runs.run[runs.begin[kb]], runs.begin[kb + 1] - runs.begin[kb], true);
  }
}

// a member alone in its run is an ordinary segment
int kind_in_run(int kind, const Run& run) { return (kind & 2) && run.n_segs == 1 ? kind & 1 : kind; }

bool packed_slot(const fcp_problem* p, const fcp_slot& sl) { return sl.n_pairs == 1 && (p->pairs[sl.pair_begin].kind & 2); }

// Items of two sub-tiles.
int64_t q_items_of(const fcp_problem* p, int rows) {
  return ceil_div(rows, item_rows(p)) * ((p->n_q_heads / p->n_kv_heads) % 2 == 0 ? p->n_q_heads / 2 : p->n_q_heads);
}

// A row tile of at most 64 rows may take four heads of a group of 4, 8, ..: all eight waves of the workgroup have rows then.
bool four_heads(const fcp_problem* p, int rows) { return rows <= kFwdTileM / 2 && (p->n_q_heads / p->n_kv_heads) % 4 == 0; }

// How many fewer items `rows` rows are then.
int64_t four_heads_save(const fcp_problem* p, int rows) { return four_heads(p, (rows - 1) % kFwdTileM + 1) ? p->n_q_heads / 4 : 0; }

constexpr int kFourHeadsItems = 512;     // of two heads: beyond, four always pay (see kTwoHeadsTile)

// Append KV rows to the spans of a forward segment (those from span0 on): to the last one where they follow it.
void append_span(std::vector<DevPair>* spans, int32_t span0, int32_t start, int32_t len, int kind) {
  DevPair* last = (int32_t)spans->size() > span0 ? &spans->back() : nullptr;
  if (last && last->kind == FCP_KIND_FULL && !(kind & 2) && last->kv_start + last->kv_len == start && (int64_t)last->kv_len + len <= kMaxSpan) {
    if (kind == FCP_KIND_DIAG) { last->kind = kind; last->ext = last->kv_len; }
    last->kv_len += len;
  } else {
    spans->push_back({start, len, kind, 0});
  }
}

// The spans of a pair for rows [row0, row0 + rows) of its query block: no more than kMaxSpan rows each.  Under a DIAG pair those
// rows see the columns before them in full.
void add_spans(std::vector<DevPair>* spans, int32_t span0, const KvSeg& k, int kind, int32_t row0, int32_t rows) {
  const int32_t full = kind == FCP_KIND_FULL ? k.len : kind == FCP_KIND_DIAG ? row0 : 0;
  for (int32_t off = 0, n; off < full; off += n) {
    n = std::min(full - off, kMaxSpan);
    append_span(spans, span0, k.start + off, n, FCP_KIND_FULL);
  }
  if (kind != FCP_KIND_FULL) append_span(spans, span0, k.start + full, kind == FCP_KIND_DIAG ? rows : k.len, kind);
}

}  // namespace

void expand_problem(const fcp_problem* p, bool forward_only, Expanded* x) {
  const Runs runs = make_runs(p);
  const bool spill = (p->flags & FCP_FLAG_BWD_SPILL_DS) != 0, direct = (p->flags & FCP_FLAG_DIRECT_SINGLE) != 0;
  for (int b = 0; b < p->n_kv_blocks; b++)
    for (int i = runs.begin[b]; i < runs.begin[b + 1]; i++)
      x->kv.push_back({p->kv_blocks[b].tok_start + runs.run[i].off, runs.run[i].len, runs.run[i].seq, 0, 0});
  if (p->n_segments) {
    int64_t t_q = 0;
    for (int b = 0; b < p->n_q_blocks; b++) t_q += p->q_blocks[b].tok_len;
    x->q_seg.assign(t_q, 0);
  }
  // query side: pairs (with the query rows and the KV segment each joins), forward and dQ segments
  struct Join { int32_t q_start, q_len, kv_seg; };
  std::vector<Join> joins;
  // what tables without packed blocks become at most (18749 pairs: queue builder 10.6 ms with lists grown as they fill, 6.0 so)
  x->fwd.reserve(p->n_slots);
  x->spans.reserve(p->n_pairs);
  if (!forward_only) { x->pairs.reserve(p->n_pairs); joins.reserve(p->n_pairs); x->dq.reserve(p->n_q_blocks); }
  int64_t frag = kDsSinkFrags;
  for_q_blocks(p, runs, [&](int b, int s0, int s1, const Run* run, int n_runs, bool packed) {
    const fcp_block& qb = p->q_blocks[b];
    const int to_final = (direct && s1 - s0 == 1) ? 1 : 0;
    // the pairs of a run are consecutive, for dQ
    for (int m = 0; m < n_runs; m++) {
      const int32_t q0 = qb.tok_start + run[m].off, p0 = (int32_t)x->pairs.size();
      for (int s = s0; s < s1; s++) {
        const fcp_slot& sl = p->slots[s];
        // a packed query block may have slots of FULL pairs too: the forward walks them once, with all rows of the block
        const bool whole = packed && !packed_slot(p, sl);
        if (!whole || m == 0) {
          // the forward's rows: a segment of at most kMaxSpan rows each
          const int32_t first = whole ? qb.tok_start : q0, out = sl.row_start + (whole ? 0 : run[m].off), len = whole ? qb.tok_len : run[m].len;
          for (int32_t row = 0, n; row < len; row += n) {
            n = std::min(len - row, kMaxSpan);
            const int32_t span0 = (int32_t)x->spans.size();
            for (int i = sl.pair_begin; i < sl.pair_begin + sl.n_pairs; i++) {
              const fcp_pair& pr = p->pairs[i];
              add_spans(&x->spans, span0, x->kv[runs.begin[pr.kv_blk] + ((pr.kind & 2) ? m : 0)], kind_in_run(pr.kind, run[m]), row, n);
            }
            x->fwd.push_back({first + row, n, out + row, span0, (int32_t)x->spans.size() - span0, whole ? qb.seq : run[m].seq, to_final, s - s0});
          }
        }
        if (forward_only) continue;
        for (int i = sl.pair_begin; i < sl.pair_begin + sl.n_pairs; i++) {
          const fcp_pair& pr = p->pairs[i];
          const int32_t seg = runs.begin[pr.kv_blk] + ((pr.kind & 2) ? m : 0);
          KvSeg& k = x->kv[seg];
          const int kind = kind_in_run(pr.kind, run[m]);
          x->pairs.push_back({k.start, k.len, kind, spill ? (int32_t)frag : 0});
          joins.push_back({q0, run[m].len, seg});
          k.n_deps++;
          frag += p->n_q_heads * ds_frags_per_head(kind, run[m].len, k.len);
        }
      }
      if (run[m].n_segs > 1)
        for (int i = run[m].seg_begin; i < run[m].seg_begin + run[m].n_segs; i++) {
          const int lo = p->segments[i].tok_off - run[m].off, hi = lo + p->segments[i].tok_len;
          std::fill(x->q_seg.begin() + q0 + lo, x->q_seg.begin() + q0 + hi, seg_word(lo, hi));
        }
      if (!forward_only) x->dq.push_back({q0, run[m].len, q0, p0, (int32_t)x->pairs.size() - p0, run[m].seq, 0, 0});
    }
  });
  if (forward_only) return;

  // KV side: the dependencies of each KV segment, in query order, the DIAG one last: the tiles of one KV segment then
  // walk the FULL dependencies in lockstep (identical step sequences, same XCD), so the Q / dO stream they share stays
  // in L2; they only diverge on the diagonal, where each tile starts at its own row.
  int32_t d = 0;
  for (KvSeg& k : x->kv) { k.dep_begin = d; d += k.n_deps; k.n_deps = 0; }
  x->deps.resize(x->pairs.size());
  for (size_t i = 0; i < joins.size(); i++) {
    KvSeg& k = x->kv[joins[i].kv_seg];
    x->deps[k.dep_begin + k.n_deps++] = {joins[i].q_start, joins[i].q_len, x->pairs[i].kind, x->pairs[i].ext};
  }
  for (const KvSeg& k : x->kv)
    std::stable_partition(x->deps.begin() + k.dep_begin, x->deps.begin() + k.dep_begin + k.n_deps, [](const BwdDep& e) { return !(e.kind & 1); });
}

size_t static_plan_bytes(const fcp_problem* p) {
  int64_t items = 0;
  for (int s = 0; s < p->n_slots; s++) items += q_items_of(p, p->q_blocks[p->slots[s].q_blk].tok_len);
  auto align = [](size_t x) { return (x + 255) & ~(size_t)255; };
  return 1024 + align(16 * (size_t)std::max(1, p->n_pairs)) + align(72 * (size_t)std::max<int64_t>(1, items));
}

int compute_layout(const fcp_problem* p, bool forward_only, WsLayout* L) {
  std::memset(L, 0, sizeof(*L));
  const Runs runs = make_runs(p);
  for (const Run& r : runs.run) L->n_bwd_items += ceil_div(r.len, kBwdTileN) * p->n_kv_heads;
  int64_t frags = kDsSinkFrags, fwd_save = 0, dq_save = 0;
  for_q_blocks(p, runs, [&](int b, int s0, int s1, const Run* run, int n_runs, bool packed) {
    int64_t items = 0, save = 0;
    for (int m = 0; m < n_runs; m++) { items += q_items_of(p, run[m].len); save += four_heads_save(p, run[m].len); }
    L->n_dq_items += items;
    dq_save += save;
    for (int s = s0; s < s1; s++) {
      const bool whole = packed && !packed_slot(p, p->slots[s]);
      L->n_fwd_items += whole ? q_items_of(p, p->q_blocks[b].tok_len) : items;
      fwd_save += whole ? four_heads_save(p, p->q_blocks[b].tok_len) : save;
      const int64_t n_pairs = (int64_t)p->slots[s].n_pairs * n_runs;
      if (!forward_only) L->n_pairs += n_pairs;
      if (p->block_size <= kMaxSpan) {
        L->n_spans += whole ? p->slots[s].n_pairs : n_pairs;
        continue;
      }
      for (int i = p->slots[s].pair_begin; i < p->slots[s].pair_begin + p->slots[s].n_pairs; i++)
        L->n_spans += ceil_div(p->kv_blocks[p->pairs[i].kv_blk].tok_len, kMaxSpan) * ceil_div(p->q_blocks[b].tok_len, kMaxSpan) * (whole ? 1 : n_runs);
    }
    if (!(p->flags & FCP_FLAG_BWD_SPILL_DS) || s0 == s1) return;
    for (int i = p->slots[s0].pair_begin; i < p->slots[s1 - 1].pair_begin + p->slots[s1 - 1].n_pairs; i++) {
      const fcp_pair& pr = p->pairs[i];
      for (int m = 0; m < n_runs; m++)
        frags += p->n_q_heads * ds_frags_per_head(pr.kind, run[m].len, runs.run[runs.begin[pr.kv_blk] + ((pr.kind & 2) ? m : 0)].len);
    }
  });
  L->fwd_four_save = fwd_save;
  L->dq_four_save = dq_save;
  const bool few_fwd = fwd_save > 0 && L->n_fwd_items <= kFourHeadsItems, few_dq = !forward_only && dq_save > 0 && L->n_dq_items <= kFourHeadsItems;
  L->n_fwd_items -= fwd_save;
  L->n_dq_items -= dq_save;
  if (few_fwd || few_dq) choose_split(p, forward_only, L);      // may go back to two heads, so before anything is laid out
  std::vector<int32_t> slots_of(p->n_q_blocks, 0);
  for (int s = 0; s < p->n_slots; s++) slots_of[p->slots[s].q_blk]++;
  const bool direct = (p->flags & FCP_FLAG_DIRECT_SINGLE) != 0;
  {
    // Chunk of the merge: small enough for kMergeMinItems work items (the kernel walks the slots of a chunk one
    // after the other, so a few long items leave most of the chip idle), a multiple of 32 entries, at most kMergeChunk.
    int64_t entries = 0;
    for (int b = 0; b < p->n_q_blocks; b++)
      if (!(direct && slots_of[b] == 1)) entries += (int64_t)p->q_blocks[b].tok_len * p->n_q_heads;
    L->merge_chunk = (int)std::min<int64_t>(kMergeChunk, std::max<int64_t>(32, ceil_div(ceil_div(entries, kMergeMinItems), 32) * 32));
  }
  for (int b = 0; b < p->n_q_blocks; b++) {
    if (!(direct && slots_of[b] == 1))
      L->n_merge_items += ceil_div((int64_t)p->q_blocks[b].tok_len * p->n_q_heads, L->merge_chunk);
    L->t_q += p->q_blocks[b].tok_len;
  }
  if (L->t_q * p->n_q_heads > INT32_MAX) { set_error("more than 2^31-1 (query row, head) entries"); return FCP_ERR_UNSUPPORTED; }
  if (std::max(L->n_pairs, L->n_spans) > INT32_MAX || L->n_fwd_items > INT32_MAX || L->n_bwd_items > INT32_MAX || L->n_merge_items > INT32_MAX || L->n_dq_items > INT32_MAX) {
    set_error("too many pairs or work items"); return FCP_ERR_UNSUPPORTED;
  }
  auto align = [](size_t x) { return (x + 255) & ~(size_t)255; };
  size_t off = align(sizeof(WsHeader));
  L->off_pairs = off;       if (!forward_only) off = align(off + sizeof(DevPair) * (size_t)std::max<int64_t>(1, L->n_pairs));
  L->off_fwd_items = off;   off = align(off + sizeof(QItem) * (size_t)std::max<int64_t>(1, L->n_fwd_items));
  L->off_q_seg = off;       off = align(off + (p->n_segments ? sizeof(uint16_t) * (size_t)L->t_q : 0));
  if (!forward_only) {
    L->off_bwd_deps = off;    off = align(off + sizeof(BwdDep) * (size_t)std::max<int64_t>(1, L->n_pairs));
    L->off_bwd_items = off;   off = align(off + sizeof(BwdItem) * (size_t)std::max<int64_t>(1, L->n_bwd_items));
    L->off_merge_items = off; off = align(off + sizeof(MergeItem) * (size_t)std::max<int64_t>(1, L->n_merge_items));
    L->off_slot_rh = off;     off = align(off + sizeof(int32_t) * (size_t)std::max(1, p->n_slots));
    L->off_dq_items = off;    off = align(off + sizeof(QItem) * (size_t)std::max<int64_t>(1, L->n_dq_items));
  }
  // last of the tables: there are usually far fewer spans than the layout has room for, and only those are uploaded (4142 pairs,
  // 257 spans, 16 heads: queue builder 406 us with all of the room, 387 so; forward without a workspace 163 and 151)
  L->off_spans = off;       off = align(off + sizeof(DevPair) * (size_t)std::max<int64_t>(1, L->n_spans));
  // backward scratch, head-major [Hq][T_q] fp32: D * scale, then LSE * log2(e)
  L->off_dls = off;         off = align(off + sizeof(float) * (size_t)std::max<int64_t>(1, L->t_q * p->n_q_heads));
  L->off_lse2 = off;        off = align(off + sizeof(float) * (size_t)std::max<int64_t>(1, L->t_q * p->n_q_heads));
  L->off_ds = off;
  if (p->flags & FCP_FLAG_BWD_SPILL_DS) {
    frags++;   // the dQ kernel requests the fragments of a whole tile in pairs: one past the last may be named (never used)
    if (frags > INT32_MAX) { set_error("FCP_FLAG_BWD_SPILL_DS: more than 2^31-1 dS fragments"); return FCP_ERR_UNSUPPORTED; }
    L->n_ds_frags = frags;
    off = align(off + (size_t)frags * kDsFragBytes);
  }
  L->total = off;
  return FCP_OK;
}

namespace {

// What a launch takes, in microseconds on 256 compute units, whole (one workgroup walks an item's tiles or steps one after the
// other) and split (fwd_split_kernel, bwd_split_kernel).  Forward and dQ: least-squares fits to 1300 to 1600 random problems a kernel and head
// size, each run in both forms: 1 to 60 sequences, whole ones and only their last blocks, 1 to 128 heads, chains of 1 to 360 tiles.  Root mean square
// error 8 to 12 % (whole) and 11 to 15 % (split).  dK/dV: fits to 58 shapes, which chose well on 2838 such problems too.
// whole:  the start, and an end: dK/dV the longest item or the mean load and a time per item; forward and dQ every item on the compute unit
//         that is free first.  An item in which at most half of the waves have rows walks its tiles faster.
// split:  a start, the work, a time per workgroup (unit: 8, dK/dV 4) and the longest chain, which is an eighth; workgroups past the rows of
//         their item cost too.  Each 32 rows read K and V by themselves, which takes longer the less of all K / V stays in the caches (stream:
//         that many times as long at 312 MB more).
struct LaunchCost { double whole, tile, item, half, split, split_tile, split_unit, split_chain, split_empty, stream_most, gain; };
constexpr LaunchCost kLaunchCost[2][3] = {      // [d = 128][forward, dQ, dK/dV]
    {{0.7, 0.98, 6.9, 0.70, 3.9, 1.34, 10.6, 0.177, 1.04, 2.0, 1.05},
     {0.5, 1.39, 7.0, 0.74, 3.9, 1.63, 9.6, 0.258, 1.27, 0.8, 1.05},
     {6.4, 0.538, 5.8, 1.0, 5.1, 0.470, 5.8, 0.143, 0.22, 0.0, 1.15}},
    {{0.0, 1.30, 9.1, 0.65, 4.3, 2.74, 29.2, 0.246, 2.60, 2.0, 1.05},
     {0.0, 2.00, 10.0, 0.74, 4.2, 3.65, 28.7, 0.368, 3.16, 0.8, 1.05},
     {7.2, 0.703, 10.0, 1.0, 4.6, 0.948, 25.7, 0.194, 1.38, 0.0, 1.15}}};
// gain: split only what gains that much by the fits.  Of 5906 forward and dQ launches 31 are then slower than whole by more than 3 % (30 % at most),
// of 2838 of dK/dV 37 (12 %); all in all they take 0.5 % more than with the faster form of each.
constexpr double kStreamBytes = 312e6;
constexpr int kSplitMaxItems = 512;      // two to a compute unit: the fits reach no further, and walking larger tables would cost

// A row tile of at most 64 rows: four heads to an item make half as many items, whose tiles take longer, since all eight waves have rows
// instead of four.  With more than kFourHeadsItems items of two heads it always pays; below, it depends on how the items come out on the compute
// units.  Two heads / four, us: 176 items of 48 tiles (the last 64 rows of 65600 tokens, 16/4 heads, d = 128) 51 / 71, 320 of 32 tiles 47 / 52,
// dQ of 256 items of 65 tiles 127 / 138; 320 of one tile (sequences of 64) 18.2 / 13.7, 160 of one 11.5 / 11.1.
constexpr double kFourHeadsGain = 1.02;        // else two: where both come out even, two were up to 7 % the faster
constexpr double kForwardGroup = 0.012;        // what each workgroup adds to the start of a forward, us

// The items of one kernel.  Their tiles (steps): of the longest, of all; `units`: their 32-row units as fractions of a full item's.
struct LaunchLoad {
  int64_t longest = 0, tiles = 0, items = 0;
  double unit_tiles = 0, units = 0;
  struct Chains { int64_t tiles, count; bool half, four; };
  std::vector<Chains> chains;     // forward and dQ
  void add(int64_t n, int64_t count, double share) {
    longest = std::max(longest, n); tiles += n * count; items += count;
    unit_tiles += n * count * share; units += count * share;
  }
  // The whole launch, the longest items first; those of four heads as such, or as two of two each.
  double makespan(const LaunchCost& c, bool four) const {
    auto two = [&](const Chains& k) { return k.four && !four; };
    auto cost = [&](const Chains& k) { return c.item + c.tile * k.tiles * (two(k) || k.half ? c.half : 1.0); };
    int64_t n = 0;
    double last = 0;
    for (const Chains& k : chains) { n += two(k) ? 2 * k.count : k.count; last = std::max(last, cost(k)); }
    if (n > kCus) {
      std::vector<double> x;
      for (const Chains& k : chains) x.insert(x.end(), two(k) ? 2 * k.count : k.count, cost(k));
      std::sort(x.begin(), x.end(), std::greater<double>());
      std::priority_queue<double, std::vector<double>, std::greater<double>> free_at(std::greater<double>(), std::vector<double>(x.begin(), x.begin() + kCus));
      for (int64_t i = kCus; i < n; i++) {
        const double t = free_at.top() + x[i];
        free_at.pop();
        free_at.push(t);
        last = std::max(last, t);
      }
    }
    return c.whole + last;
  }
  int64_t groups(bool four) const {       // workgroups of the whole launch
    int64_t n = 0;
    for (const Chains& k : chains) n += k.four && !four ? 2 * k.count : k.count;
    return std::min<int64_t>(n, kCus);
  }
  // times: makespan with items of two heads and of four
  bool four_pays(const double times[2], double per_group) const {
    return times[0] + per_group * groups(false) > kFourHeadsGain * (times[1] + per_group * groups(true));
  }
  // full: units of a full item; most: workgroups that an item gets
  double split(const LaunchCost& c, int full, int most, double kv_bytes) const {
    const double stream = 1 + std::min(c.stream_most, kv_bytes / kStreamBytes), empty = (double)items * most - units * full;
    return c.split + c.split_tile * unit_tiles / kCus * stream + c.split_unit * units / kCus + c.split_chain * longest + c.split_empty * empty / kCus;
  }
  static constexpr int kCus = 256;
};

}  // namespace

namespace {

// Every slot holds all KV blocks that its rows see: no query block's result is merged from several.
bool slots_complete(const fcp_problem* p) {
  auto seq_of = [&](int kv_blk) { return kv_blk >= 0 && kv_blk < p->n_kv_blocks ? p->kv_blocks[kv_blk].seq : -1; };
  for (int s = 0; s < p->n_slots; s++) {
    const fcp_slot& sl = p->slots[s];
    if (sl.n_pairs == 0) continue;
    const fcp_pair &first = p->pairs[sl.pair_begin], &last = p->pairs[sl.pair_begin + sl.n_pairs - 1];
    if (seq_of(first.kv_blk - 1) == seq_of(first.kv_blk) || (!(last.kind & 1) && seq_of(last.kv_blk + 1) == seq_of(last.kv_blk))) return false;
  }
  return true;
}

// 32-row units of the forward if every KV block of a query block's sequence were a slot of its own.
int64_t units_by_blocks(const fcp_problem* p) {
  std::unordered_map<int32_t, int64_t> blocks_of;
  for (int i = 0; i < p->n_kv_blocks; i++) blocks_of[p->kv_blocks[i].seq]++;
  int64_t units = 0;
  for (int b = 0; b < p->n_q_blocks; b++) units += ceil_div(p->q_blocks[b].tok_len, 32) * p->n_q_heads * blocks_of[p->q_blocks[b].seq];
  return units;
}

}  // namespace

void choose_split(const fcp_problem* p, bool forward_only, WsLayout* L) {
  if (L->chosen) return;
  const LaunchCost* cost = kLaunchCost[p->head_dim == 128];
  const int G = p->n_q_heads / p->n_kv_heads, heads = G % 2 == 0 ? p->n_q_heads / 2 : p->n_q_heads, rows_of_item = item_rows(p);
  // The forward is chosen from its own tables alone, so that fcp_block_attn_fwd_static and a workspace choose alike.  Partial slots go
  // further: the two kernels round P to bf16 against different references, so the stages of a plan and its one-pass forward agree to fp32
  // rounding only where all of them take the same one.  What they have in common are the blocks, not the items of one launch.  At 2.5 (1)
  // units to a compute unit a launch of the shortest slots takes what a whole one does.
  const int64_t most_units = p->head_dim == 128 ? 256 : 640;
  const bool spill = (p->flags & FCP_FLAG_BWD_SPILL_DS) != 0;
  bool fit_fwd = false;
  if (L->n_fwd_items > 0 && L->n_fwd_items <= std::max<int64_t>(kSplitMaxItems, most_units)) {
    // a planned block has no more slots than its sequence has KV blocks, so items are no more than units; others may have any number
    if (!slots_complete(p)) L->split_fwd = L->n_fwd_items <= most_units && units_by_blocks(p) <= most_units;
    else fit_fwd = L->n_fwd_items <= kSplitMaxItems;
  }
  const bool query = !forward_only && L->n_dq_items <= kSplitMaxItems, keys = !forward_only && L->n_bwd_items <= kSplitMaxItems;
  const bool may_two_fwd = !L->four_settled && L->four_fwd() && L->n_fwd_items + L->fwd_four_save <= kFourHeadsItems;
  const bool may_two_dq = !L->four_settled && !forward_only && L->four_dq() && L->n_dq_items + L->dq_four_save <= kFourHeadsItems;
  L->four_settled = true;
  if (p->flags & FCP_FLAG_WHOLE_ITEMS && !may_two_fwd && !may_two_dq) { L->split_fwd = false; return; }
  if (!L->split_fwd && !fit_fwd && !query && !keys && !may_two_fwd) return;
  LaunchLoad fwd, dq, dkdv;
  const Runs runs = make_runs(p);
  std::vector<int64_t> steps(keys ? runs.run.size() : 0, 0);     // of a KV segment's dependencies that it sees in full
  std::vector<char> diag(keys ? runs.run.size() : 0, 0);         // it has one that it sees from its own rows on
  int max_fwd = 0, max_dq = 0, max_kv = 0;
  auto segment = [&](LaunchLoad* l, bool four_on, bool keep, int* most, int64_t full, int64_t diag_cols, int len) {
    *most = std::max(*most, len);
    for (int64_t row = 0; row < len; row += rows_of_item) {          // len: up to 2^31 - 1
      const int n = (int)std::min<int64_t>(rows_of_item, len - row);
      const int64_t tiles = ceil_div(full + std::min<int64_t>(diag_cols, row + n), kQTileN);
      const int four = four_on && four_heads(p, n) ? 2 : 1;
      l->add(tiles, heads / four, (double)ceil_div(n, 32) * 32 * four / rows_of_item);
      if (keep) l->chains.push_back({tiles, heads / four, four == 1 && n <= rows_of_item / 2, four == 2});
    }
  };
  for_q_blocks(p, runs, [&](int b, int s0, int s1, const Run* run, int n_runs, bool packed) {
    for (int m = 0; m < n_runs; m++) {
      int64_t dq_full = 0, dq_diag = 0;
      for (int s = s0; s < s1; s++) {
        const fcp_slot& sl = p->slots[s];
        const bool whole = packed && !packed_slot(p, sl);
        int64_t full = 0, diag_cols = 0;
        for (int i = sl.pair_begin; i < sl.pair_begin + sl.n_pairs; i++) {
          const fcp_pair& pr = p->pairs[i];
          const int seg = runs.begin[pr.kv_blk] + ((pr.kind & 2) ? m : 0);
          ((pr.kind & 1) ? diag_cols : full) += runs.run[seg].len;
          if (!keys) continue;
          if (pr.kind & 1) diag[seg] = 1; else steps[seg] += ceil_div(run[m].len, 32) * G;
        }
        if (!whole || m == 0) segment(&fwd, L->four_fwd(), may_two_fwd || fit_fwd, &max_fwd, full, diag_cols, whole ? p->q_blocks[b].tok_len : run[m].len);
        dq_full += full; dq_diag += diag_cols;
      }
      segment(&dq, L->four_dq(), may_two_dq || query, &max_dq, dq_full, dq_diag, run[m].len);
    }
  });
  // units of a sub-tile, and of an item: two sub-tiles (one, where odd groups have no second row tile), or four heads of two units or one
  auto units_of = [&](bool four, int most) {
    const int per_tile = (int)ceil_div(std::min(most, kFwdTileM), 32);
    if (four) return most > kFwdTileM / 2 ? SplitUnits{8, 4} : SplitUnits{4 * per_tile, per_tile};
    return SplitUnits{per_tile * (G % 2 == 0 || most > kFwdTileM ? 2 : 1), per_tile};
  };
  L->fwd_units = units_of(L->four_fwd(), max_fwd);
  L->dq_units = units_of(L->four_dq(), max_dq);
  double kv_bytes = 0;
  for (int i = 0; i < p->n_kv_blocks; i++) kv_bytes += 4.0 * p->kv_blocks[i].tok_len * p->n_kv_heads * p->head_dim;
  double fwd_whole[2] = {0, 0}, dq_whole[2] = {0, 0};      // with items of two heads, of four
  for (int four = 0; four < 2; four++) {
    fwd_whole[four] = four && !L->four_fwd() ? fwd_whole[0] : fwd.makespan(cost[0], four);
    dq_whole[four] = four && !L->four_dq() ? dq_whole[0] : dq.makespan(cost[1], four);
  }
  if (fit_fwd) L->split_fwd = std::min(fwd_whole[0], fwd_whole[1]) > cost[0].gain * fwd.split(cost[0], 8, L->fwd_units.units, kv_bytes);
  double dq_time = 0;
  if (query && L->n_dq_items > 0) {
    dq_time = dq.split(cost[1], 8, L->dq_units.units, kv_bytes);
    L->split_dq = std::min(dq_whole[0], dq_whole[1]) > cost[1].gain * dq_time;
  }
  for (size_t k = 0; k < steps.size(); k++)
    for (int64_t off = 0, len = runs.run[k].len; off < len; off += kBwdTileN) {
      const int n = (int)std::min<int64_t>(kBwdTileN, len - off);
      max_kv = std::max(max_kv, n);
      dkdv.add(steps[k] + (diag[k] ? ceil_div(len - off, 32) * G : 0), p->n_kv_heads, (double)ceil_div(n, 32) * 32 / kBwdTileN);
    }
  L->split_kv_units = (int)ceil_div(max_kv, 32);
  const double whole_dkdv = cost[2].whole + cost[2].tile * std::max<double>(dkdv.longest, (double)dkdv.tiles / LaunchLoad::kCus) + cost[2].item * dkdv.items / LaunchLoad::kCus;
  const double dkdv_time = dkdv.split(cost[2], 4, L->split_kv_units, 0);
  L->split_dkdv = keys && L->n_bwd_items > 0 && whole_dkdv > cost[2].gain * dkdv_time;
  // Both in one launch behind the D pass, or dQ with D in it and then dK/dV.  The D pass walks the heads one after the other (2.9 us and 0.21 a head
  // at d = 64, twice that at 128); what one launch saves is the shorter half.  Backward of 1500 random problems, joint / one after the other: up to
  // 12 heads of d = 64 0.84, 16 and 24 heads 1.04 below 35 us and 0.91 above, 64 heads of d = 128 43 / 15 us at its worst.
  const int heads64 = p->n_q_heads * (p->head_dim / 64);
  L->joint_bwd = L->split_dq && L->split_dkdv && (heads64 <= 12 || (heads64 <= 24 && dq_time + dkdv_time > 35));
  if (p->flags & FCP_FLAG_WHOLE_ITEMS) L->joint_bwd = L->split_fwd = L->split_dq = L->split_dkdv = false;
  // Split launches keep items of four heads: the units are the same, their neighbours on an XCD share more (dQ of 256 items, d = 64 84 -> 80 us).
  const bool two_fwd = may_two_fwd && !L->split_fwd && !fwd.four_pays(fwd_whole, kForwardGroup);
  const bool two_dq = may_two_dq && (!L->split_dq || spill) && !dq.four_pays(dq_whole, 0);
  if (two_fwd) { L->n_fwd_items += L->fwd_four_save; L->fwd_four_save = 0; }
  if (two_dq) { L->n_dq_items += L->dq_four_save; L->dq_four_save = 0; }
  L->chosen = !two_fwd && !two_dq;
}

// Layouts validated by fcp_queue_build, keyed by the workspace they were built into.  A launch on that
// workspace with the same descriptor scalars reuses the layout instead of walking every table again: the
// kernels read the device copy of the tables that fcp_queue_build made, so the host tables matter to a
// launch only through their counts.  A workspace the registry does not know (or a descriptor that differs)
// takes the full validation path.
namespace {
struct LayoutKey {
  const void* workspace;
  int32_t v[11];
  bool operator==(const LayoutKey& o) const { return workspace == o.workspace && std::memcmp(v, o.v, sizeof(v)) == 0; }
};
LayoutKey make_key(const fcp_problem* p, const void* ws) {
  return LayoutKey{ws, {p->n_q_heads, p->n_kv_heads, p->head_dim, p->block_size, p->flags & (FCP_FLAG_DIRECT_SINGLE | FCP_FLAG_BWD_SPILL_DS | FCP_FLAG_WHOLE_ITEMS),
                        p->n_kv_blocks, p->n_q_blocks, p->n_pairs, p->n_slots, p->n_slot_rows, p->n_segments}};
}
constexpr int kLayoutCacheSize = 32;
std::mutex g_layout_mutex;
std::pair<LayoutKey, WsLayout> g_layout_cache[kLayoutCacheSize];
int g_layout_count = 0, g_layout_next = 0;
}  // namespace

void remember_layout(const fcp_problem* p, const void* workspace, const WsLayout& L) {
  const LayoutKey key = make_key(p, workspace);
  std::lock_guard<std::mutex> lock(g_layout_mutex);
  for (int i = 0; i < g_layout_count; i++)
    if (g_layout_cache[i].first.workspace == workspace) { g_layout_cache[i] = {key, L}; return; }
  g_layout_cache[g_layout_next] = {key, L};
  g_layout_next = (g_layout_next + 1) % kLayoutCacheSize;
  g_layout_count = std::min(g_layout_count + 1, kLayoutCacheSize);
}

int layout_for(const fcp_problem* p, const void* workspace, WsLayout* L) {
  if (p && workspace && p->softmax_scale >= 0.0f) {
    const LayoutKey key = make_key(p, workspace);
    std::lock_guard<std::mutex> lock(g_layout_mutex);
    for (int i = 0; i < g_layout_count; i++)
      if (g_layout_cache[i].first == key) { *L = g_layout_cache[i].second; return FCP_OK; }
  }
  int rc = validate_problem(p);
  if (rc) return rc;
  rc = compute_layout(p, false, L);
  if (rc == FCP_OK) choose_split(p, false, L);
  return rc;
}

namespace {

// Column of a pair (not a span: 0) or span where its DIAG block starts.
int diag_off(const DevPair& p, bool spans) { return spans ? p.ext : 0; }

// 64-row KV tiles that a query-stationary item visits: every pair (span) in full, a DIAG one up to the item's last row.
void count_tiles(QItem* it, const std::vector<DevPair>& pairs, bool spans) {
  const int row_hi = std::max(it->tile_off[0] + it->q_rows[0], it->tile_off[1] + it->q_rows[1]);
  int n = 0;
  for (int i = it->pair_begin; i < it->pair_begin + it->n_pairs; i++) {
    const int nc = (pairs[i].kind & 1) ? std::min(pairs[i].kv_len, diag_off(pairs[i], spans) + row_hi) : pairs[i].kv_len;
    n += (nc + kQTileN - 1) / kQTileN;
  }
  it->n_tiles = n;
  if (it->n_pairs > 0) it->first = pairs[it->pair_begin];
  it->diag_last = -1;
  if (it->n_pairs > 0 && (pairs[it->pair_begin + it->n_pairs - 1].kind & 1)) it->diag_last = diag_off(pairs[it->pair_begin + it->n_pairs - 1], spans);
}

int32_t chain_of(const QItem& it) { return it.n_tiles; }
int32_t chain_of(const BwdItem& it) { return it.n_iv; }

// Work items in groups that stay together: the items of a unit (one per (segment, KV head)) are consecutive in `items`, a
// group is a run of units in `order`.
template <class Item>
struct ItemGroups {
  std::vector<Item> items;
  std::vector<int32_t> unit_end;                   // items of unit u end here
  std::vector<int32_t> order, group_end;           // units by group; units of group g end here in `order`
  std::vector<int64_t> weight, key;                // per group
  // the items pushed since the last call form one more unit, for now a group of its own
  void close_unit(int64_t w, int64_t k) {
    order.push_back((int32_t)unit_end.size());
    unit_end.push_back((int32_t)items.size());
    group_end.push_back((int32_t)order.size());
    weight.push_back(w); key.push_back(k);
  }
  // XCD affinity: groups whose keys agree after division by `div` become one group (units concatenated in the order the
  // groups came; the keys are divided).  With a key per (sequence, KV head) all work that streams the K / V (forward, dQ)
  // or Q / dO (dK/dV) rows of one sequence and KV head runs on one XCD and finds them in that XCD's L2 (measured on the
  // training step: forward -1.2 %, dK/dV -0.6 %, dQ from dS -2 %).  Only done while the largest merged group stays below
  // three quarters of an XCD's fair share: a batch dominated by one sequence keeps the finer groups, which balance better.
  void merge(int64_t div) {
    const size_t n = weight.size();
    std::unordered_map<int64_t, int32_t> where;    // key -> merged group, in order of first appearance
    where.reserve(n);
    std::vector<int32_t> to(n), end2;
    std::vector<int64_t> w2, key2;
    int64_t total = 0, largest = 0;
    for (size_t i = 0; i < n; i++) {
      to[i] = where.emplace(key[i] / div, (int32_t)w2.size()).first->second;
      if (to[i] == (int32_t)w2.size()) { w2.push_back(0); key2.push_back(key[i] / div); end2.push_back(0); }
      w2[to[i]] += weight[i];
      total += weight[i];
      largest = std::max(largest, w2[to[i]]);
      end2[to[i]] += group_end[i] - (i ? group_end[i - 1] : 0);
    }
    if (largest * kNumXcd * 4 > total * 3) return;
    std::vector<int32_t> pos(end2.size());         // where the next unit of a merged group goes
    for (size_t g = 0, at = 0; g < end2.size(); g++) { pos[g] = (int32_t)at; at += end2[g]; end2[g] = (int32_t)at; }
    std::vector<int32_t> order2(order.size());
    for (size_t i = 0; i < n; i++)
      for (int32_t u = i ? group_end[i - 1] : 0; u < group_end[i]; u++) order2[pos[to[i]]++] = order[u];
    order.swap(order2); group_end.swap(end2); weight.swap(w2); key.swap(key2);
  }
  // Longest-processing-time assignment of weighted groups to the XCD queues: groups in
  // descending weight, each to the currently lightest queue.  Ties resolve to the lower index.  out: room for all items.
  // split: for a split kernel, which has no queues (workgroup b runs on XCD b % 8): the longest chains first, by turns on the XCDs
  // (the last workgroups of 4000 tokens, 4 heads, d = 64 started 4.7 of 10.5 us late, whole chains before them; forward 10.8 -> 9.2 us).
  void spread_over_xcds(Item* out, int32_t begin[kNumXcd + 1], bool split) const {
    std::vector<int> by_weight(weight.size());
    std::iota(by_weight.begin(), by_weight.end(), 0);
    std::stable_sort(by_weight.begin(), by_weight.end(), [&](int a, int b) { return weight[a] > weight[b]; });
    std::vector<int> per_xcd[kNumXcd];
    int64_t load[kNumXcd] = {0};
    for (int g : by_weight) {
      const int best = (int)(std::min_element(load, load + kNumXcd) - load);
      per_xcd[best].push_back(g);
      load[best] += weight[g];
    }
    Item* const first = out;
    for (int x = 0; x < kNumXcd; x++) {
      begin[x] = (int32_t)(out - first);
      for (int g : per_xcd[x])
        for (int32_t u = g ? group_end[g - 1] : 0; u < group_end[g]; u++) {
          const int32_t unit = order[u];
          out = std::copy(items.begin() + (unit ? unit_end[unit - 1] : 0), items.begin() + unit_end[unit], out);
        }
    }
    begin[kNumXcd] = (int32_t)(out - first);
    if (split) std::stable_sort(first, out, [](const Item& a, const Item& b) { return chain_of(a) > chain_of(b); });
  }
};

// The query-stationary items (forward, dQ) of a list of segments, one unit per (segment, KV head): its items share
// K/V.  An item joins two sub-tiles: heads (2j, 2j+1) of the group on one row tile when G is even, else row tiles
// (2j, 2j+1) of one head; with `four`, of a row tile of at most 64 rows heads 4j .. 4j + 3 when G is a multiple of 4.  out: n_items of them; false if there would be another number.
bool q_items(const fcp_problem* p, const std::vector<QSeg>& segs, const std::vector<DevPair>& pairs, bool spans, bool four, bool split, int64_t n_items, QItem* out,
             int32_t begin[kNumXcd + 1]) {
  const int G = p->n_q_heads / p->n_kv_heads, heads_per_item = G % 2 == 0 ? 2 : 1;
  ItemGroups<QItem> groups;
  groups.items.reserve(n_items);
  std::vector<int64_t> tile_w;
  std::vector<QItem> rows;                        // the segment's items but for their heads
  int64_t n_ord = 1;
  for (const QSeg& sg : segs) n_ord = std::max<int64_t>(n_ord, sg.ordinal + 1);
  for (const QSeg& sg : segs) {
    const int n_tiles = (int)ceil_div(sg.len, kFwdTileM);
    tile_w.assign(n_tiles, 0);
    for (int t = 0; t < n_tiles; t++) {
      const int off = t * kFwdTileM, n_rows = std::min(kFwdTileM, sg.len - off);
      for (int i = sg.pair_begin; i < sg.pair_begin + sg.n_pairs; i++)
        tile_w[t] += (int64_t)n_rows * ((pairs[i].kind & 1) ? std::min(pairs[i].kv_len, diag_off(pairs[i], spans) + off + n_rows) : pairs[i].kv_len);
    }
    rows.clear();
    int64_t w = 0;                                // of the segment and one KV head
    // later tiles of a DIAG pair are heavier: they come first
    for (int t = n_tiles - 1; t >= 0; t -= G % 2 == 0 ? 1 : 2) {
      QItem it{};
      it.pair_begin = sg.pair_begin; it.n_pairs = sg.n_pairs; it.to_final = sg.to_final; it.q_blk_len = sg.len;
      for (int k = 0; k < 2; k++) {
        const bool absent = G % 2 != 0 && k == 1 && t == 0;      // no second sub-tile: row 0 of the first, no rows
        const int tile = G % 2 != 0 && k == 1 && t > 0 ? t - 1 : t, off = tile * kFwdTileM;
        it.q_start[k] = sg.start + off; it.q_rows[k] = absent ? 0 : std::min(kFwdTileM, sg.len - off);
        it.out_row[k] = sg.out_row + off; it.tile_off[k] = off;
        if (!absent) w += tile_w[tile] * (G / heads_per_item);
      }
      count_tiles(&it, pairs, spans);
      rows.push_back(it);
    }
    for (int g = 0; g < p->n_kv_heads; g++) {
      for (const QItem& r : rows) {
        const int heads = four && four_heads(p, r.q_rows[0]) ? 4 : heads_per_item;
        for (int hh = 0; hh < G; hh += heads) {
          groups.items.push_back(r);
          groups.items.back().head[0] = g * G + hh; groups.items.back().head[1] = g * G + hh + heads - 1;
        }
      }
      groups.close_unit(w, ((int64_t)sg.seq * p->n_kv_heads + g) * n_ord + sg.ordinal);
    }
  }
  // First the slots that cover the same KV range of a sequence (the r-th slot of each of its query blocks), then the
  // whole sequence: the workgroups of an XCD then walk one KV range at a time, which stays in that XCD's L2, instead of
  // as many ranges as a query block has slots (forward of 13000 rows at the end of a 200000-token sequence, 16 KV heads,
  // slots of 4096 columns, plus 118000 tokens of short sequences: 11.2 -> 9.7 ms).
  if ((int64_t)groups.items.size() != n_items) return false;
  groups.merge(1);
  groups.merge(n_ord);
  groups.spread_over_xcds(out, begin, split);
  return true;
}

}  // namespace
}  // namespace fcp

using namespace fcp;

extern "C" const char* fcp_last_error(void) { return g_err; }

extern "C" int fcp_plan_blocks(const int32_t* seq_lens, int32_t n_seqs, int32_t block_size,
                               int32_t causal, int32_t coalesce,
                               const int32_t* q_owned, int32_t n_q_owned,
                               fcp_block* kv_blocks, int32_t* n_kv_blocks,
                               fcp_block* q_blocks, int32_t* n_q_blocks,
                               fcp_pair* pairs, int32_t* n_pairs,
                               fcp_slot* slots, int32_t* n_slots,
                               int32_t* n_slot_rows) {
  if (n_seqs < 0 || (n_seqs > 0 && !seq_lens) || block_size <= 0 || coalesce < 0 || n_q_owned < 0 ||
      !n_kv_blocks || !n_q_blocks || !n_pairs || !n_slots || !n_slot_rows) {
    set_error("fcp_plan_blocks: invalid argument"); return FCP_ERR_INVALID_ARG;
  }
  // Pass 1: per-sequence block counts and offsets.
  std::vector<int64_t> first_blk(n_seqs + 1, 0), tok_off(n_seqs + 1, 0);
  for (int s = 0; s < n_seqs; s++) {
    if (seq_lens[s] < 0) { set_error("fcp_plan_blocks: seq_lens[%d] < 0", s); return FCP_ERR_INVALID_ARG; }
    first_blk[s + 1] = first_blk[s] + ceil_div(seq_lens[s], block_size);
    tok_off[s + 1] = tok_off[s] + seq_lens[s];
  }
  if (tok_off[n_seqs] > INT32_MAX || first_blk[n_seqs] > INT32_MAX) {
    set_error("fcp_plan_blocks: more than 2^31-1 tokens or blocks"); return FCP_ERR_UNSUPPORTED;
  }
  auto nblk = [&](int s) { return (int32_t)(first_blk[s + 1] - first_blk[s]); };
  auto blk_len = [&](int s, int i) { return std::min<int32_t>(block_size, seq_lens[s] - i * block_size); };
  const int64_t need_kv = first_blk[n_seqs];
  // Owned query blocks.
  const bool all_owned = (q_owned == nullptr);
  if (!all_owned) {
    for (int t = 0; t < n_q_owned; t++) {
      const int32_t s = q_owned[2 * t], i = q_owned[2 * t + 1];
      if (s < 0 || s >= n_seqs || i < 0 || i >= nblk(s)) {
        set_error("fcp_plan_blocks: q_owned[%d] = (%d, %d) out of range", t, s, i); return FCP_ERR_INVALID_ARG;
      }
      if (t > 0) {
        const int32_t ps = q_owned[2 * t - 2], pi = q_owned[2 * t - 1];
        if (ps > s || (ps == s && pi >= i)) {
          set_error("fcp_plan_blocks: q_owned must be strictly increasing in (seq, idx)");
          return FCP_ERR_INVALID_ARG;
        }
      }
    }
  }
  const int64_t need_q = all_owned ? need_kv : n_q_owned;
  // Pass 2: counts of pairs, slots, partial rows.
  int64_t need_pairs = 0, need_slots = 0, need_rows = 0;
  auto for_each_owned = [&](auto&& fn) {
    if (all_owned) {
      for (int s = 0; s < n_seqs; s++)
        for (int i = 0; i < nblk(s); i++) fn(s, i);
    } else {
      for (int t = 0; t < n_q_owned; t++) fn(q_owned[2 * t], q_owned[2 * t + 1]);
    }
  };
  for_each_owned([&](int s, int i) {
    const int64_t np = causal ? (i + 1) : nblk(s);
    const int64_t ns = coalesce == 0 ? 1 : ceil_div(np, coalesce);
    need_pairs += np;
    need_slots += ns;
    need_rows += ns * blk_len(s, i);
  });
  if (need_pairs > INT32_MAX || need_rows > INT32_MAX) {
    set_error("fcp_plan_blocks: more than 2^31-1 pairs or partial rows"); return FCP_ERR_UNSUPPORTED;
  }
  const int32_t cap_kv = *n_kv_blocks, cap_q = *n_q_blocks, cap_p = *n_pairs, cap_s = *n_slots;
  *n_kv_blocks = (int32_t)need_kv; *n_q_blocks = (int32_t)need_q; *n_pairs = (int32_t)need_pairs;
  *n_slots = (int32_t)need_slots; *n_slot_rows = (int32_t)need_rows;
  if (!kv_blocks && !q_blocks && !pairs && !slots) return FCP_OK;   // size query
  if (!kv_blocks || !q_blocks || !pairs || !slots) {
    set_error("fcp_plan_blocks: pass all four tables or none"); return FCP_ERR_INVALID_ARG;
  }
  if (cap_kv < need_kv || cap_q < need_q || cap_p < need_pairs || cap_s < need_slots) {
    set_error("fcp_plan_blocks: table capacity too small (need %lld kv, %lld q, %lld pairs, %lld slots)",
              (long long)need_kv, (long long)need_q, (long long)need_pairs, (long long)need_slots);
    return FCP_ERR_BUFFER_TOO_SMALL;
  }
  // Pass 3: fill.
  for (int s = 0; s < n_seqs; s++)
    for (int i = 0; i < nblk(s); i++)
      kv_blocks[first_blk[s] + i] = {s, i, (int32_t)(tok_off[s] + (int64_t)i * block_size), blk_len(s, i)};
  int32_t qb = 0, qtok = 0, np_out = 0, ns_out = 0, row = 0;
  for_each_owned([&](int s, int i) {
    const int32_t len = blk_len(s, i);
    q_blocks[qb] = {s, i, qtok, len};
    qtok += len;
    const int32_t np = causal ? (i + 1) : nblk(s);
    for (int32_t r = 0; r < np; r++) {
      const bool opens = (coalesce == 0) ? (r == 0) : (r % coalesce == 0);
      if (opens) {
        slots[ns_out] = {qb, np_out, 0, row};
        ns_out++;
        row += len;
      }
      const int32_t kind = (causal && r == i) ? FCP_KIND_DIAG : FCP_KIND_FULL;
      pairs[np_out] = {qb, (int32_t)(first_blk[s] + r), kind, ns_out - 1};
      slots[ns_out - 1].n_pairs++;
      np_out++;
    }
    qb++;
  });
  return FCP_OK;
}

extern "C" int fcp_plan_blocks_packed(const int32_t* seq_lens, int32_t n_seqs, int32_t block_size,
                                      int32_t causal, int32_t coalesce,
                                      const int32_t* q_owned, int32_t n_q_owned,
                                      const int32_t* unit_of_block,
                                      fcp_block* kv_blocks, int32_t* n_kv_blocks,
                                      fcp_block* q_blocks, int32_t* n_q_blocks,
                                      fcp_pair* pairs, int32_t* n_pairs,
                                      fcp_slot* slots, int32_t* n_slots,
                                      int32_t* n_slot_rows,
                                      fcp_segment* segments, int32_t* n_segments) {
  if (n_seqs < 0 || (n_seqs > 0 && !seq_lens) || block_size <= 0 || coalesce < 0 || n_q_owned < 0 ||
      !n_kv_blocks || !n_q_blocks || !n_pairs || !n_slots || !n_slot_rows || !n_segments) {
    set_error("fcp_plan_blocks_packed: invalid argument"); return FCP_ERR_INVALID_ARG;
  }
  // The unpacked table: block u of it is (u_seq[u], u_idx[u]) with u_len[u] tokens.
  std::vector<int32_t> u_seq, u_idx, u_len, first_u(n_seqs + 1, 0);
  for (int s = 0; s < n_seqs; s++) {
    if (seq_lens[s] < 0) { set_error("fcp_plan_blocks_packed: seq_lens[%d] < 0", s); return FCP_ERR_INVALID_ARG; }
    const int64_t nb = ceil_div(seq_lens[s], block_size);
    if ((int64_t)u_seq.size() + nb > INT32_MAX) { set_error("fcp_plan_blocks_packed: more than 2^31-1 blocks"); return FCP_ERR_UNSUPPORTED; }
    for (int i = 0; i < nb; i++) {
      u_seq.push_back(s); u_idx.push_back(i);
      u_len.push_back(std::min<int32_t>(block_size, seq_lens[s] - i * block_size));
    }
    first_u[s + 1] = (int32_t)u_seq.size();
  }
  const int32_t nu = (int32_t)u_seq.size();
  if (nu > 0 && !unit_of_block) { set_error("fcp_plan_blocks_packed: unit_of_block is NULL"); return FCP_ERR_INVALID_ARG; }
  // Units: size, lowest member, summed length; a multi-block unit is a packed block led by its lowest member.
  std::vector<int32_t> u_count(nu, 0), u_lead(nu, -1), u_last(nu, -1), next_member(nu, -1);
  std::vector<int64_t> u_sum(nu, 0);
  for (int u = 0; u < nu; u++) {
    const int32_t g = unit_of_block[u];
    if (g < 0 || g >= nu) { set_error("fcp_plan_blocks_packed: unit_of_block[%d] = %d out of range", u, g); return FCP_ERR_INVALID_ARG; }
    if (u_count[g]++ == 0) u_lead[g] = u; else next_member[u_last[g]] = u;
    u_last[g] = u;
    u_sum[g] += u_len[u];
  }
  for (int u = 0; u < nu; u++) {
    const int32_t g = unit_of_block[u];
    if (u_count[g] < 2) continue;
    if (u_idx[u] != 0 || first_u[u_seq[u] + 1] - first_u[u_seq[u]] != 1 || u_len[u] >= block_size) {
      set_error("fcp_plan_blocks_packed: block %d shares unit %d but is not a whole sequence shorter than a block", u, g);
      return FCP_ERR_INVALID_ARG;
    }
    if (u_sum[g] > block_size) { set_error("fcp_plan_blocks_packed: unit %d does not fit into one block", g); return FCP_ERR_INVALID_ARG; }
  }
  auto packed = [&](int u) { return u_count[unit_of_block[u]] >= 2; };
  auto leads = [&](int u) { return !packed(u) || u_lead[unit_of_block[u]] == u; };
  // Ownership per unpacked block.
  std::vector<char> own(nu, q_owned ? 0 : 1);
  if (q_owned) {
    for (int t = 0; t < n_q_owned; t++) {
      const int32_t s = q_owned[2 * t], i = q_owned[2 * t + 1];
      if (s < 0 || s >= n_seqs || i < 0 || i >= first_u[s + 1] - first_u[s]) {
        set_error("fcp_plan_blocks_packed: q_owned[%d] = (%d, %d) out of range", t, s, i); return FCP_ERR_INVALID_ARG;
      }
      if (t > 0 && (q_owned[2 * t - 2] > s || (q_owned[2 * t - 2] == s && q_owned[2 * t - 1] >= i))) {
        set_error("fcp_plan_blocks_packed: q_owned must be strictly increasing in (seq, idx)"); return FCP_ERR_INVALID_ARG;
      }
      own[first_u[s] + i] = 1;
    }
    for (int u = 0; u < nu; u++)
      if (packed(u) && own[u] != own[u_lead[unit_of_block[u]]]) {
        set_error("fcp_plan_blocks_packed: unit %d is owned in part", unit_of_block[u]); return FCP_ERR_INVALID_ARG;
      }
  }
  // Counts.
  int64_t need_kv = 0, need_q = 0, need_pairs = 0, need_slots = 0, need_rows = 0, need_seg = 0, tokens = 0;
  for (int u = 0; u < nu; u++) {
    tokens += u_len[u];
    if (packed(u)) need_seg++;
    if (!leads(u)) continue;
    need_kv++;
    if (!own[u]) continue;
    need_q++;
    const int64_t len = packed(u) ? u_sum[unit_of_block[u]] : u_len[u];
    const int64_t np = packed(u) ? 1 : (causal ? u_idx[u] + 1 : first_u[u_seq[u] + 1] - first_u[u_seq[u]]);
    const int64_t ns = coalesce == 0 ? 1 : ceil_div(np, coalesce);
    need_pairs += np; need_slots += ns; need_rows += ns * len;
  }
  if (tokens > INT32_MAX || need_pairs > INT32_MAX || need_rows > INT32_MAX) {
    set_error("fcp_plan_blocks_packed: more than 2^31-1 tokens, pairs or partial rows"); return FCP_ERR_UNSUPPORTED;
  }
  const int32_t cap_kv = *n_kv_blocks, cap_q = *n_q_blocks, cap_p = *n_pairs, cap_s = *n_slots, cap_g = *n_segments;
  *n_kv_blocks = (int32_t)need_kv; *n_q_blocks = (int32_t)need_q; *n_pairs = (int32_t)need_pairs;
  *n_slots = (int32_t)need_slots; *n_slot_rows = (int32_t)need_rows; *n_segments = (int32_t)need_seg;
  if (!kv_blocks && !q_blocks && !pairs && !slots && !segments) return FCP_OK;   // size query
  if (!kv_blocks || !q_blocks || !pairs || !slots || (need_seg > 0 && !segments)) {
    set_error("fcp_plan_blocks_packed: pass all tables or none"); return FCP_ERR_INVALID_ARG;
  }
  if (cap_kv < need_kv || cap_q < need_q || cap_p < need_pairs || cap_s < need_slots || cap_g < need_seg) {
    set_error("fcp_plan_blocks_packed: table capacity too small (need %lld kv, %lld q, %lld pairs, %lld slots, %lld segments)",
              (long long)need_kv, (long long)need_q, (long long)need_pairs, (long long)need_slots, (long long)need_seg);
    return FCP_ERR_BUFFER_TOO_SMALL;
  }
  // Fill: KV blocks and segments first (a pair needs the new index of an unpacked block), then the owned side.
  std::vector<int32_t> kv_of(nu, -1);
  int32_t nk = 0, ng = 0, tok = 0;
  for (int u = 0; u < nu; u++) {
    if (!leads(u)) continue;
    int32_t len = u_len[u];
    if (packed(u)) {
      len = 0;
      for (int m = u; m >= 0; m = next_member[m]) {     // members in ascending unpacked order; the lead is the lowest
        segments[ng++] = {nk, u_seq[m], len, u_len[m]};
        len += u_len[m];
      }
    }
    kv_of[u] = nk;
    kv_blocks[nk++] = {u_seq[u], packed(u) ? 0 : u_idx[u], tok, len};
    tok += len;
  }
  int32_t nq = 0, qtok = 0, np_out = 0, ns_out = 0, row = 0;
  for (int u = 0; u < nu; u++) {
    if (!leads(u) || !own[u]) continue;
    const fcp_block& kb = kv_blocks[kv_of[u]];
    q_blocks[nq] = {kb.seq, kb.idx, qtok, kb.tok_len};
    qtok += kb.tok_len;
    if (packed(u)) {
      slots[ns_out] = {nq, np_out, 1, row};
      pairs[np_out++] = {nq, kv_of[u], causal ? FCP_KIND_PACKED_DIAG : FCP_KIND_PACKED_FULL, ns_out};
      ns_out++;
      row += kb.tok_len;
    } else {
      const int32_t s = u_seq[u], i = u_idx[u];
      const int32_t np = causal ? (i + 1) : first_u[s + 1] - first_u[s];
      for (int32_t r = 0; r < np; r++) {
        if ((coalesce == 0) ? (r == 0) : (r % coalesce == 0)) {
          slots[ns_out++] = {nq, np_out, 0, row};
          row += kb.tok_len;
        }
        pairs[np_out++] = {nq, kv_of[first_u[s] + r], (causal && r == i) ? FCP_KIND_DIAG : FCP_KIND_FULL, ns_out - 1};
        slots[ns_out - 1].n_pairs++;
      }
    }
    nq++;
  }
  return FCP_OK;
}

extern "C" int fcp_stage_tables(const fcp_pair* pairs, int32_t n_pairs, const fcp_slot* slots, int32_t n_slots,
                                const fcp_block* q_blocks, int32_t n_q_blocks, int32_t stage,
                                fcp_pair* stage_pairs, int32_t* n_stage_pairs, fcp_slot* stage_slots, int32_t* n_stage_slots,
                                int32_t* n_stages) {
  if (n_pairs < 0 || n_slots < 0 || n_q_blocks < 0 || stage < 0 || (n_pairs && !pairs) || (n_slots && !slots) ||
      (n_q_blocks && !q_blocks) || !n_stage_pairs || !n_stage_slots || !n_stages) {
    set_error("fcp_stage_tables: invalid argument"); return FCP_ERR_INVALID_ARG;
  }
  // pass 1: the stage-th slot of every query block (slots of a block are consecutive), counts
  int64_t need_pairs = 0, need_slots = 0;
  int32_t most = 0;
  for (int s = 0, local = 0; s < n_slots; s++) {
    const fcp_slot& sl = slots[s];
    if (sl.q_blk < 0 || sl.q_blk >= n_q_blocks || sl.pair_begin < 0 || sl.n_pairs < 0 || (int64_t)sl.pair_begin + sl.n_pairs > n_pairs ||
        (s > 0 && sl.q_blk < slots[s - 1].q_blk)) {
      set_error("fcp_stage_tables: slots[%d] is inconsistent", s); return FCP_ERR_INVALID_ARG;
    }
    local = (s > 0 && slots[s - 1].q_blk == sl.q_blk) ? local + 1 : 0;
    most = std::max(most, local + 1);
    if (local == stage) { need_slots++; need_pairs += sl.n_pairs; }
  }
  const int32_t cap_p = *n_stage_pairs, cap_s = *n_stage_slots;
  *n_stage_pairs = (int32_t)need_pairs; *n_stage_slots = (int32_t)need_slots; *n_stages = most;
  if (!stage_pairs && !stage_slots) return FCP_OK;
  if (!stage_pairs || !stage_slots) { set_error("fcp_stage_tables: pass both tables or none"); return FCP_ERR_INVALID_ARG; }
  if (cap_p < need_pairs || cap_s < need_slots) {
    set_error("fcp_stage_tables: table capacity too small (need %lld pairs, %lld slots)", (long long)need_pairs, (long long)need_slots);
    return FCP_ERR_BUFFER_TOO_SMALL;
  }
  int32_t np = 0, ns = 0;
  for (int s = 0, local = 0; s < n_slots; s++) {
    const fcp_slot& sl = slots[s];
    local = (s > 0 && slots[s - 1].q_blk == sl.q_blk) ? local + 1 : 0;
    if (local != stage) continue;
    stage_slots[ns] = {sl.q_blk, np, sl.n_pairs, q_blocks[sl.q_blk].tok_start};
    for (int i = sl.pair_begin; i < sl.pair_begin + sl.n_pairs; i++)
      stage_pairs[np++] = {pairs[i].q_blk, pairs[i].kv_blk, pairs[i].kind, ns};
    ns++;
  }
  return FCP_OK;
}

extern "C" int fcp_workspace_bytes(const fcp_problem* p, size_t* bytes) {
  if (!bytes) { set_error("fcp_workspace_bytes: bytes is NULL"); return FCP_ERR_INVALID_ARG; }
  int rc = validate_problem(p);
  if (rc) return rc;
  WsLayout L;
  rc = compute_layout(p, false, &L);
  if (rc) return rc;
  *bytes = L.total;
  return FCP_OK;
}

// The host image of the workspace sections that the kernels read: header (zeroed counters, queue
// ranges, zero / +inf pages), spans, forward items and, unless forward_only, the pairs, the backward,
// dQ and merge tables.  `image` is resized to what there is of them: up to the last span.
int fcp::build_queue_image(const fcp_problem* p, const Expanded& x, const WsLayout& L, bool forward_only, std::vector<unsigned char>* image) {
  if ((int64_t)x.spans.size() > L.n_spans) { set_error("internal: span count mismatch"); return FCP_ERR_INVALID_ARG; }
  image->assign(L.off_spans + x.spans.size() * sizeof(DevPair), 0);
  std::vector<unsigned char>& host = *image;
  WsHeader* hdr = reinterpret_cast<WsHeader*>(host.data());
  for (float& v : hdr->infs) v = INFINITY;
  auto put = [&](size_t off, const auto& v) { if (!v.empty()) std::memcpy(host.data() + off, v.data(), v.size() * sizeof(v[0])); };
  if ((int64_t)x.pairs.size() != L.n_pairs) { set_error("internal: pair count mismatch"); return FCP_ERR_INVALID_ARG; }
  put(L.off_pairs, x.pairs);
  put(L.off_spans, x.spans);
  put(L.off_q_seg, x.q_seg);
  if (!q_items(p, x.fwd, x.spans, true, L.four_fwd(), L.split_fwd, L.n_fwd_items, reinterpret_cast<QItem*>(host.data() + L.off_fwd_items), hdr->fwd_begin)) {
    set_error("internal: forward item count mismatch"); return FCP_ERR_INVALID_ARG;
  }
  if (forward_only) return FCP_OK;
  // ---- dQ: query-stationary items over all pairs of a query segment; with dS kept dq_ds_kernel draws them from the queues, whatever dQ alone would take
  if (!q_items(p, x.dq, x.pairs, false, L.four_dq(), L.split_dq && !(p->flags & FCP_FLAG_BWD_SPILL_DS), L.n_dq_items, reinterpret_cast<QItem*>(host.data() + L.off_dq_items), hdr->dq_begin)) {
    set_error("internal: dQ item count mismatch"); return FCP_ERR_INVALID_ARG;
  }
  // ---- dK / dV: dependency lists per KV segment, one group per (KV segment, KV head)
  {
    const int G = p->n_q_heads / p->n_kv_heads;
    put(L.off_bwd_deps, x.deps);
    ItemGroups<BwdItem> groups;
    groups.items.reserve(L.n_bwd_items);
    std::vector<int64_t> tile_w, tile_steps;
    for (const KvSeg& k : x.kv) {
      const int n_tiles = (int)ceil_div(k.len, kBwdTileN);
      tile_w.assign(n_tiles, 0);
      tile_steps.assign(n_tiles, 0);
      for (int t = 0; t < n_tiles; t++) {
        const int off = t * kBwdTileN, rows = std::min(kBwdTileN, k.len - off);
        for (int i = k.dep_begin; i < k.dep_begin + k.n_deps; i++) {
          const int q_rows = (x.deps[i].kind & 1) ? std::max(0, x.deps[i].q_len - off) : x.deps[i].q_len;   // off is a multiple of 32
          tile_w[t] += (int64_t)rows * G * q_rows;
          tile_steps[t] += G * ceil_div(q_rows, 32);
        }
        if (tile_steps[t] + 3 > INT32_MAX) { set_error("too many steps in a backward work item"); return FCP_ERR_UNSUPPORTED; }
      }
      const int64_t w = std::accumulate(tile_w.begin(), tile_w.end(), (int64_t)0);
      for (int g = 0; g < p->n_kv_heads; g++) {
        for (int t = 0; t < n_tiles; t++) {            // earlier tiles of a DIAG pair are heavier
          const int off = t * kBwdTileN;
          groups.items.push_back({k.start + off, std::min(kBwdTileN, k.len - off), off, k.dep_begin, k.n_deps, g, k.len, (int32_t)((tile_steps[t] + 3) & ~1),
                                  k.n_deps > 0 ? x.deps[k.dep_begin] : BwdDep{0, 0, 0, 0}});
        }
        groups.close_unit(w, (int64_t)k.seq * p->n_kv_heads + g);
      }
    }
    groups.merge(1);
    if ((int64_t)groups.items.size() != L.n_bwd_items) { set_error("internal: backward item count mismatch"); return FCP_ERR_INVALID_ARG; }
    groups.spread_over_xcds(reinterpret_cast<BwdItem*>(host.data() + L.off_bwd_items), hdr->bwd_begin, L.split_dkdv);
  }
  // ---- merge: row-head chunks per query block; slots of a query block are consecutive.
  {
    std::vector<int32_t> slot_begin(p->n_q_blocks + 1, 0);
    for (int s = 0; s < p->n_slots; s++) slot_begin[p->slots[s].q_blk + 1]++;
    for (int b = 0; b < p->n_q_blocks; b++) slot_begin[b + 1] += slot_begin[b];
    int32_t* slot_rh = reinterpret_cast<int32_t*>(host.data() + L.off_slot_rh);
    for (int s = 0; s < p->n_slots; s++) {
      const int64_t rh = (int64_t)p->slots[s].row_start * p->n_q_heads;
      if (rh > INT32_MAX) { set_error("partial buffers exceed 2^31-1 (row, head) entries"); return FCP_ERR_UNSUPPORTED; }
      slot_rh[s] = (int32_t)rh;
    }
    MergeItem* mi = reinterpret_cast<MergeItem*>(host.data() + L.off_merge_items);
    int64_t n = 0;
    for (int b = 0; b < p->n_q_blocks; b++) {
      const fcp_block& qb = p->q_blocks[b];
      if ((p->flags & FCP_FLAG_DIRECT_SINGLE) && slot_begin[b + 1] - slot_begin[b] == 1) continue;   // written by the forward
      const int64_t total = (int64_t)qb.tok_len * p->n_q_heads;
      for (int64_t off = 0; off < total; off += L.merge_chunk) {
        mi[n++] = {(int32_t)((int64_t)qb.tok_start * p->n_q_heads + off), (int32_t)std::min<int64_t>(L.merge_chunk, total - off),
                   slot_begin[b], slot_begin[b + 1] - slot_begin[b], (int32_t)off, 0, 0, 0};
      }
    }
    if (n != L.n_merge_items) { set_error("internal: merge item count mismatch"); return FCP_ERR_INVALID_ARG; }
  }
  return FCP_OK;
}

extern "C" int fcp_queue_build(const fcp_problem* p, void* workspace, size_t workspace_bytes, void* stream) {
  int rc = validate_problem(p);
  if (rc) return rc;
  WsLayout L;
  rc = compute_layout(p, false, &L);
  if (rc) return rc;
  if (!workspace || ((uintptr_t)workspace & 255)) {
    set_error("fcp_queue_build: workspace is NULL or not 256-byte aligned"); return FCP_ERR_INVALID_ARG;
  }
  if (workspace_bytes < L.total) {
    set_error("fcp_queue_build: workspace too small (%zu < %zu)", workspace_bytes, L.total);
    return FCP_ERR_BUFFER_TOO_SMALL;
  }
  choose_split(p, false, &L);
  Expanded x;
  expand_problem(p, false, &x);
  std::vector<unsigned char> host;
  rc = build_queue_image(p, x, L, false, &host);
  if (rc) return rc;
  hipError_t e = hipMemcpyAsync(workspace, host.data(), host.size(), hipMemcpyHostToDevice, (hipStream_t)stream);
  if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);
  if (e != hipSuccess) { set_error("fcp_queue_build: %s", hipGetErrorString(e)); return FCP_ERR_HIP; }
  remember_layout(p, workspace, L);
  return FCP_OK;
}

extern "C" int fcp_launch_probe(const fcp_problem* p, int32_t forward_only, int32_t info[17]) {
  if (!info) { set_error("fcp_launch_probe: info is NULL"); return FCP_ERR_INVALID_ARG; }
  int rc = validate_problem(p);
  if (rc) return rc;
  WsLayout L;
  rc = compute_layout(p, forward_only != 0, &L);
  if (rc) return rc;
  choose_split(p, forward_only != 0, &L);
  const int32_t head[8] = {L.split_fwd, L.split_dq, L.split_dkdv, (int32_t)L.n_fwd_items, (int32_t)L.n_dq_items, (int32_t)L.n_bwd_items, L.four_fwd(), L.four_dq()};
  std::fill(std::copy(head, head + 8, info), info + 16, 0);
  info[16] = L.joint_bwd;
  if (forward_only) return FCP_OK;
  Expanded x;
  expand_problem(p, false, &x);
  std::vector<unsigned char> image;
  rc = build_queue_image(p, x, L, false, &image);
  if (rc) return rc;
  const WsHeader* hdr = reinterpret_cast<const WsHeader*>(image.data());
  const QItem* items = reinterpret_cast<const QItem*>(image.data() + L.off_dq_items);
  for (int q = 0; q < kNumXcd; q++)
    for (int32_t i = hdr->dq_begin[q]; i < hdr->dq_begin[q + 1]; i++) info[8 + q] += items[i].n_tiles;
  return FCP_OK;
}
