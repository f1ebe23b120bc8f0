// Host-side work list of the paged decode-attention kernel.
#pragma once

#include <stdint.h>

#include <vector>

#include "kernels/kernels.hpp"

namespace hxf {

// One decoding sequence: batch entry, context length (the query attends to tokens
// [0, ctx)) and its block table on the host (at least ceil(ctx / 16) pages; null:
// the sequence is never grouped with others).
struct DecodeSeq {
  int entry;
  int ctx;
  const int32_t* pages;
  int n_pages = 1 << 30;   // entries of the table, where ctx may exceed it (a plan alone may be asked for)
};

struct DecodePlan {
  std::vector<DecodeItem> items;    // one-tile items, then the n_wide two-tile items (each longest first)
  int64_t n_items = 0, n_wide = 0;
  std::vector<MergeItem> merges;    // one per (sequence, kv-head), in sequence order
  int64_t n_parts = 0;              // partial slots used
  int64_t kv_tokens = 0;            // (token, kv-head) pairs read: the sum of the item lengths

  // the planner's working memory, kept so that a plan used again allocates nothing
  struct Stream {
    int32_t first, len;       // tokens [first, first + len)
    int32_t rows, n_rows;     // sequences served: members[rows .. rows + n_rows)
    int32_t piece, n_pieces;  // tokens per piece (the last may be shorter)
    int32_t slot_off;         // offset of this stream's pieces inside each row's slot block
  };
  struct Run {                // the pieces of a stream that have one length
    int32_t len, stream, piece0, n;
  };
  std::vector<Stream> streams;
  std::vector<Run> runs;
  std::vector<uint64_t> order;
  std::vector<int32_t> members, shared, slots, base;
};

// Sequences whose block tables start with the same physical pages (forks of one
// retained parent share its full pages) form a group.  The shared full pages are
// attended by items that serve up to decode_rows_wide(G) of the group's sequences at
// once (two-tile items when more than decode_rows_narrow(G)), so each shared page is
// read once per such item instead of once per sequence; every sequence's own pages
// get items of their own.  All streams are
// cut into equal page-aligned partitions sized to fill the resident wavefronts
// (decode_target_tokens), and the partials of a (sequence, kv-head) occupy
// consecutive slots, merged by log-sum-exp.
void plan_decode(const std::vector<DecodeSeq>& seqs, int hkv, int G, DecodePlan& out);
// The same in two steps, for a caller that has the items written where they are uploaded from:
// everything but `items` (left as it is), then the n_items records.
void plan_decode_streams(const std::vector<DecodeSeq>& seqs, int hkv, int G, DecodePlan& out);
void write_decode_items(const DecodePlan& plan, const std::vector<DecodeSeq>& seqs, int hkv, DecodeItem* items);

// Chunked-prefill work list.  Each (prefill entry, kv-head, block of qpi queries) is
// one item over the key tiles its queries see.  With fewer items than CUs, an item
// longer than the per-slot share of one pass over the resident workgroups (at least
// kPrefillMinTiles) is cut into equal key ranges whose partials a merge job combines.
// Items are launched most tiles first, the long and short ones of the first pass
// paired on the CUs.
struct PrefillEntry {
  int entry, pos0, n;   // batch entry, position of its first query, queries
};
struct PrefillPlan {
  std::vector<PrefillItem> items;
  std::vector<PrefillMerge> merges;
  int64_t n_parts = 0;
  int64_t tiles = 0;    // key tiles over all items
};
void plan_prefill(const std::vector<PrefillEntry>& entries, int hkv, int qpi, PrefillPlan& out);
// Partial slots the prefill plan of n_items items can use (split items only).
inline int64_t prefill_parts_bound(int64_t n_items) { return n_items + kPrefillResident; }

// Upper bound of partial slots (and items) for n sequences of at most max_ctx tokens.
inline int64_t decode_parts_bound(int64_t n_seqs, int64_t hkv, int64_t max_ctx) {
  return n_seqs * hkv * ((max_ctx + kDecodeMinPartition - 1) / kDecodeMinPartition + 1);
}

}  // namespace hxf
