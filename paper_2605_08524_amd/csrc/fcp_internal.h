// Internal layout shared by the host scheduler and the HIP kernels (not part of the ABI).
#ifndef FCP_INTERNAL_H_
#define FCP_INTERNAL_H_

#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "fcp.h"

namespace fcp {

constexpr int kNumXcd = 8;          // MI355X: 8 XCDs, each with its own L2; workgroup b runs on XCD b % 8
constexpr int kFwdTileM = 128;      // query rows per query-stationary work item (4 waves x 32 rows)
constexpr int kBwdTileN = 128;      // KV rows per backward work item (4 waves x 32 rows)
constexpr int kMergeChunk = 1024;   // most (row, head) entries per merge work item (fewer when there is little to merge)
constexpr int kMergeMinItems = 2048;  // the merge aims at this many work items at least: 8 per compute unit

// Device-side records (all int32 so the host can build them as plain arrays).
// A packed block reaches the kernels cut into runs of whole members, each a query (KV) segment with one pair of its own
// (expand_problem).  Neighbours join a run while it fits the rows of one query-stationary item; its pair keeps the PACKED
// kind and the kernels mask by member (q_seg).  A member alone in its run is an ordinary segment: FULL or DIAG, no mask.
// Forward, GQA 32/8, d = 128, 1024-token blocks, when runs replaced one segment per member, against that and against the block
// walked whole with the union of its rows' key ranges, on one box: 2048 sequences of 8 tokens 105 us (821, 164); 49152 tokens in
// sequences of 16-256: 335 us (365, 477).
// ext: first 32x32 dS fragment of the pair in the spill buffer (FCP_FLAG_BWD_SPILL_DS; else 0).
// The forward walks spans instead: neighbouring pairs of a slot whose KV rows follow each other, joined (FULL ones, and the DIAG
// one that ends them).  Its tiles then run on across block borders, and what the walk looks up per pair is looked up once
// per slot.  ext of a span: column where its DIAG block starts.
struct DevPair { int32_t kv_start, kv_len, kind, ext; };
// Rows of a span, and of a forward segment (QSeg): the forward holds 4 * (columns of a span) in 32 bits.  Whole items.
constexpr int32_t kMaxSpan = 1 << 28;
static_assert(kMaxSpan % (2 * kFwdTileM) == 0, "a query block in segments has as many items as in one");
// Query-stationary item of two 128-row sub-tiles that walk the same pair list and share a KV head
// (two query heads of a group, or two neighbouring row tiles of one head; q_rows[1] = 0: none).  head[1] = head[0] + 3: four heads
// of a group on one row tile of at most 64 rows, wave w: head w / 2.  With two heads half of the waves had no rows there: sequences of
// 16-256 tokens, 32/8 heads, d = 128, 49152 of them in shared blocks, forward 308 -> 288 us, training step of 65536 1705 -> 1656.
// to_final != 0 (forward items only): the slot is the only one of its query block.
// q_blk_len (dQ items only): rows of the whole query block (of the member, in a packed block).
// n_tiles: 64-row KV tiles the item walks (a DIAG pair only up to the item's last query row).
// pair_begin, n_pairs, first, diag_last: spans in forward items, pairs in dQ items.
// first: the first of its pairs (in the record, so that an item's first tile needs no second table read).
// diag_last: column of the last span where its DIAG block starts, -1 if it has none (a wave whose rows end early need not compute
// the tiles past them).
struct QItem { int32_t q_start[2], q_rows[2], out_row[2], tile_off[2], head[2], pair_begin, n_pairs, to_final, q_blk_len, n_tiles, diag_last; DevPair first; };
constexpr int kQTileN = 64;         // KV rows per LDS tile of the query-stationary kernels
struct BwdDep  { int32_t q_start, q_len, kind, ds_frag; };
// n_iv: barrier intervals of the item: its 32-row steps (dependencies x query heads of the group; a DIAG dependency from the
// tile's own rows on) plus two of pipeline fill, rounded up to even.  first: the first of its dependencies.
struct BwdItem { int32_t kv_start, kv_rows, tile_off, dep_begin, n_deps, kv_head, kv_blk_len, n_iv; BwdDep first; };
constexpr int kMaxPackedBlock = 65535;   // tokens of a packed block: what fcp_workspace_bytes and the calls on a problem accept
// q_seg, per Q-buffer row of a joined run: first row of the row's member in the low byte, its last in the high byte, both
// counted from the run's first row (the run's KV rows have the same bounds).  A run has at most 256 rows.
inline uint16_t seg_word(int lo, int hi) { return (uint16_t)(lo | (hi - 1) << 8); }

// The dS spill buffer (FCP_FLAG_BWD_SPILL_DS) is a sequence of 2 KB fragments, one per (pair, query head,
// 32 query rows, 32 KV rows).  Fragments [0, kDsSinkFrags) take the stores of steps that have no fragment
// (pipeline fill, tiles above the diagonal); a pair's fragments follow from its ds_frag, head-major, then by
// 32-row query group; a FULL pair keeps ceil(kv_len / 32) fragments per query group, a DIAG pair only those at or
// below the diagonal (query group i keeps i + 1); a joined run keeps what FULL / DIAG keep, with zeros between members.
constexpr int kDsFragBytes = 2048;
constexpr int kDsSinkFrags = 256;
inline int64_t ds_frags_per_head(int kind, int q_len, int kv_len) {
  const int64_t nq = (q_len + 31) / 32, nk = (kv_len + 31) / 32;
  return (kind & 1) ? nq * (nq + 1) / 2 : nq * nk;   // DIAG and PACKED_DIAG: at or below the diagonal
}
struct MergeItem { int32_t out_rh, n_rh, slot_begin, n_slots, rh_off, pad0, pad1, pad2; };

// Header at the start of the workspace.  Counters are zero between launches: the last
// workgroup of a persistent launch to run dry clears the ones it used.  Every counter, every `done` and every range table has
// a 128-byte line of its own: the workgroups of a launch draw their first tickets together, and draws on one line wait for
// each other (4000 tokens, 4 heads, d = 64, forward: 21.0 us with the counters side by side, 20.2 us apart; training step
// of 16384 tokens, 16 heads, d = 64: 676 and 656).
constexpr int kCounterStride = 32;
struct WsHeader {
  int32_t fwd_counter[kNumXcd * kCounterStride];
  int32_t bwd_counter[kNumXcd * kCounterStride];
  int32_t dq_counter[kNumXcd * kCounterStride];
  int32_t fwd_done, pad0[31], bwd_done, pad1[31], dq_done, pad2[31];
  int32_t fwd_begin[kNumXcd + 1];   // item range of each XCD queue
  int32_t pad3[kCounterStride - kNumXcd - 1];
  int32_t bwd_begin[kNumXcd + 1];
  int32_t pad4[kCounterStride - kNumXcd - 1];
  int32_t dq_begin[kNumXcd + 1];
  int32_t pad5[kCounterStride - kNumXcd - 1];
  int32_t zeros[64];                // 256-byte zero page: source of LDS-DMA loads past a ragged end
  float infs[64];                   // +inf page: LSE of query rows past a ragged end (their P is 0)
};

// Workgroups of an item in a split launch at most (32 rows each), and of a sub-tile.
struct SplitUnits { int units, per_tile; };

// Byte offsets of the workspace sections, a pure function of the problem's counts.
struct WsLayout {
  int64_t n_fwd_items, n_bwd_items, n_merge_items, n_dq_items, n_pairs, n_spans, t_q;   // n_spans: at most
  int merge_chunk;  // (row, head) entries per merge work item, chosen per problem
  int64_t fwd_four_save, dq_four_save;   // how many fewer items there are because row tiles of at most 64 rows take four heads; 0: they take two
  bool four_settled;        // a choice already made stands: the sections are laid out for it
  bool chosen;              // choose_split has nothing left to do
  bool four_fwd() const { return fwd_four_save > 0; }
  bool four_dq() const { return dq_four_save > 0; }
  // choose_split: which launches go to the split kernels, and the 32-row units that an item has there at most
  bool split_fwd, split_dq, split_dkdv;
  bool joint_bwd;   // fcp_block_attn_bwd runs split dQ and dK/dV in one launch
  SplitUnits fwd_units, dq_units;
  int split_kv_units;
  int64_t n_ds_frags;   // fragments of the dS spill buffer, sinks and one fragment of slack included (0 without the flag)
  size_t off_pairs, off_spans, off_fwd_items, off_q_seg, off_bwd_deps, off_bwd_items, off_merge_items, off_slot_rh, off_dq_items, off_dls, off_lse2, off_ds, total;
};

// The problem as the kernels see it.  Segment = rows that share a pair list: a query block (KV block), or one run of
// a packed one.  ordinal: which slot of its query block a forward segment is (0 for dQ).
struct QSeg { int32_t start, len, out_row, pair_begin, n_pairs, seq, to_final, ordinal; };   // rows in the Q buffer / partial buffers
struct KvSeg { int32_t start, len, seq, dep_begin, n_deps; };
struct Expanded {
  std::vector<DevPair> pairs, spans;
  std::vector<QSeg> fwd, dq;       // per slot; per query block (all pairs of its slots)
  std::vector<KvSeg> kv;
  std::vector<BwdDep> deps;        // by KV segment
  std::vector<uint16_t> q_seg;     // per Q-buffer row (empty without packed blocks)
};
// forward_only: for an image without backward tables (pairs, dq, deps stay out)
void expand_problem(const fcp_problem* p, bool forward_only, Expanded* x);   // host; p has been validated
int validate_problem(const fcp_problem* p);           // host; sets the error text
int compute_layout(const fcp_problem* p, bool forward_only, WsLayout* L);   // host; counts only, p has been validated
void choose_split(const fcp_problem* p, bool forward_only, WsLayout* L);    // host; after compute_layout
// the layout of a problem on a workspace: from the registry that fcp_queue_build fills, else validated and computed
int layout_for(const fcp_problem* p, const void* workspace, WsLayout* L);   // host
void remember_layout(const fcp_problem* p, const void* workspace, const WsLayout& L);
// what limits fcp_block_attn_fwd_static: 1 KB, 16 bytes per pair and 72 per forward item of the plan's query blocks as given
size_t static_plan_bytes(const fcp_problem* p);
void set_error(const char* fmt, ...);
int build_queue_image(const fcp_problem* p, const Expanded& x, const WsLayout& L, bool forward_only, std::vector<unsigned char>* image);  // host

}  // namespace fcp
#endif
