// Attention work lists: decode (prefix groups, partitions, partial slots) and
// chunked prefill (query blocks, key-range splits).
#include "decode_plan.hpp"

#include <algorithm>
#include <cstring>

namespace hxf {

// The plan of a batch is rebuilt for every call (and every engine iteration), so its host time
// is on the path: whole runs of equal pieces are sorted instead of the 96-byte items, which are
// written once, in their launch order, where they are uploaded from; shared pages are compared
// as memory; the working memory is the plan's own.  Up to the items, on one host core: 64
// sequences x 8 kv-heads (1760 items) 119 -> 6 us, 256 forks of 32 prompts (4096 items) 335 -> 25.
void plan_decode_streams(const std::vector<DecodeSeq>& seqs, int hkv, int G, DecodePlan& out) {
  // every field is overwritten: the caller reuses one plan across iterations, and a stale
  // count of wide items with no items behind it would send the two-tile kernel past them
  // (the lists are resized, not cleared first: clearing would have resize() fill them)
  out.n_parts = 0;
  out.kv_tokens = 0;
  out.n_items = out.n_wide = 0;
  out.runs.clear();
  const int n = (int)seqs.size();
  if (n == 0) {
    out.merges.clear();
    return;
  }
  const int R1 = decode_rows_narrow(G), R = decode_rows_wide(G);
  auto& streams = out.streams;
  auto& members = out.members;
  streams.clear();
  members.clear();
  out.shared.assign(n, 0);

  // prefix groups: equal first page, shared length = the shortest common run of full pages;
  // one stream per R sequences of a group (in sequence order)
  auto& order = out.order;   // (first page, sequence)
  order.clear();
  for (int i = 0; i < n; ++i)
    if (seqs[i].pages) order.push_back((uint64_t)(uint32_t)seqs[i].pages[0] << 32 | (uint32_t)i);
  std::sort(order.begin(), order.end());
  const int n_known = (int)order.size();
  for (int i = 0; i < n_known;) {
    int j = i + 1;
    while (j < n_known && order[j] >> 32 == order[i] >> 32) ++j;
    if (j - i >= 2) {
      const DecodeSeq& lead = seqs[(uint32_t)order[i]];
      int s = lead.ctx / kPage;
      for (int k = i + 1; k < j && s > 0; ++k) {
        const DecodeSeq& m = seqs[(uint32_t)order[k]];
        s = std::min(s, m.ctx / kPage);
        // as memory inside both tables; a context longer than its table reads no further than the
        // first difference
        const int whole = std::min({s, m.n_pages, lead.n_pages});
        int c = std::memcmp(m.pages, lead.pages, (size_t)whole * sizeof(int32_t)) == 0 ? whole : 0;
        while (c < s && m.pages[c] == lead.pages[c]) ++c;
        s = c;
      }
      if (s > 0) {
        for (int c = i; c < j; c += R) {
          const int rows = (int)members.size();
          for (int k = c; k < std::min(j, c + R); ++k) {
            const int m = (int)(uint32_t)order[k];
            members.push_back(m);
            out.shared[m] = s * kPage;
          }
          streams.push_back({0, s * kPage, rows, (int)members.size() - rows, 0, 0, 0});
        }
      }
    }
    i = j;
  }
  // then every sequence's own tokens
  for (int i = 0; i < n; ++i)
    if (seqs[i].ctx > out.shared[i]) {
      streams.push_back({out.shared[i], seqs[i].ctx - out.shared[i], (int)members.size(), 1, 0, 0, 0});
      members.push_back(i);
    }
  int64_t total = 0;
  for (const auto& st : streams) total += st.len;
  const int64_t target = decode_target_tokens(total, (int64_t)streams.size(), hkv);

  // pieces per stream; slot blocks per sequence (shared pieces first, then own pieces)
  out.slots.assign(n, 0);
  for (size_t k = 0; k < streams.size(); ++k) {
    auto& st = streams[k];
    st.piece = decode_part_len(st.len, target);
    st.n_pieces = (st.len + st.piece - 1) / st.piece;
    st.slot_off = out.slots[members[st.rows]];
    for (int r = 0; r < st.n_rows; ++r) out.slots[members[st.rows + r]] += st.n_pieces;
    const int last = st.len - (st.n_pieces - 1) * st.piece;
    const int whole = last == st.piece ? st.n_pieces : st.n_pieces - 1;
    if (whole > 0) out.runs.push_back({st.piece, (int)k, 0, whole});
    if (whole < st.n_pieces) out.runs.push_back({last, (int)k, whole, 1});
    out.n_items += (int64_t)hkv * st.n_pieces;
    if (st.n_rows > R1) out.n_wide += (int64_t)hkv * st.n_pieces;
    out.kv_tokens += (int64_t)hkv * st.len;
  }
  out.base.resize(n);   // slot of (sequence i, kv-head 0); kv-head h adds h * slots[i]
  int64_t slot = 0;
  out.merges.resize((size_t)n * hkv);
  MergeItem* mg = out.merges.data();
  for (int i = 0; i < n; ++i) {
    out.base[i] = (int32_t)slot;
    for (int h = 0; h < hkv; ++h) {
      *mg++ = MergeItem{seqs[i].entry, h, (int32_t)slot, out.slots[i]};
      slot += out.slots[i];
    }
  }
  out.n_parts = slot;
  // Launch order: one-tile items, then the wide ones, each longest first, so that the
  // wavefronts that start last, when the chip drains, are the short pieces; equal lengths in
  // stream order.
  std::sort(out.runs.begin(), out.runs.end(), [&](const DecodePlan::Run& x, const DecodePlan::Run& y) {
    const bool wx = streams[x.stream].n_rows > R1, wy = streams[y.stream].n_rows > R1;
    if (wx != wy) return wy;
    if (x.len != y.len) return x.len > y.len;
    return x.stream != y.stream ? x.stream < y.stream : x.piece0 < y.piece0;
  });
}

void write_decode_items(const DecodePlan& plan, const std::vector<DecodeSeq>& seqs, int hkv, DecodeItem* it) {
  for (const auto& run : plan.runs) {
    const auto& st = plan.streams[run.stream];
    const int32_t* rows = plan.members.data() + st.rows;
    DecodeItem proto{};
    proto.n_rows = st.n_rows;
    int32_t first[kDecodeRows], step[kDecodeRows];
    for (int r = 0; r < kDecodeRows; ++r) {
      const int i = rows[std::min(r, st.n_rows - 1)];
      proto.entry[r] = seqs[i].entry;
      first[r] = plan.base[i] + st.slot_off + run.piece0;
      step[r] = plan.slots[i];
    }
    for (int h = 0; h < hkv; ++h) {
      proto.kvh = h;
      for (int p = 0; p < run.n; ++p, ++it) {
        proto.t0 = st.first + (run.piece0 + p) * st.piece;
        proto.t1 = proto.t0 + run.len;
        for (int r = 0; r < kDecodeRows; ++r) proto.part[r] = first[r] + p;
        *it = proto;
      }
      for (int r = 0; r < kDecodeRows; ++r) first[r] += step[r];
    }
  }
}

void plan_decode(const std::vector<DecodeSeq>& seqs, int hkv, int G, DecodePlan& out) {
  plan_decode_streams(seqs, hkv, G, out);
  out.items.resize((size_t)out.n_items);
  write_decode_items(out, seqs, hkv, out.items.data());
}

void plan_prefill(const std::vector<PrefillEntry>& entries, int hkv, int qpi, PrefillPlan& out) {
  out.items.clear();
  out.merges.clear();
  out.n_parts = 0;
  out.tiles = 0;
  std::vector<PrefillItem> whole;
  for (const PrefillEntry& e : entries)
    for (int h = 0; h < hkv; ++h)
      for (int q0 = 0; q0 < e.n; q0 += qpi) {
        const int nq = std::min(qpi, e.n - q0);
        const int t1 = (e.pos0 + q0 + nq + 31) / 32;
        whole.push_back(PrefillItem{e.entry, h, q0, nq, 0, t1, -1, 0});
        out.tiles += t1;
      }
  // With fewer items than CUs some CUs would idle: items longer than the per-slot share
  // of one pass over the resident workgroups are cut into key ranges.  With more, they
  // are not: a CU's two resident workgroups share its matrix cores, so the one left
  // running a long item runs it faster, and cutting only adds partial writes and a merge.
  const int64_t share = std::max<int64_t>((out.tiles + kPrefillResident - 1) / kPrefillResident, kPrefillMinTiles);
  const bool split = (int64_t)whole.size() < kPrefillResident / 2;
  for (const PrefillItem& it : whole) {
    if (!split || it.t1 <= share) {
      out.items.push_back(it);
      continue;
    }
    const int np = (int)((it.t1 + share - 1) / share);
    const int len = (it.t1 + np - 1) / np;
    const int part0 = (int)out.n_parts;
    int k = 0;
    for (int t0 = 0; t0 < it.t1; t0 += len, ++k) {
      PrefillItem p = it;
      p.t0 = t0;
      p.t1 = std::min(it.t1, t0 + len);
      p.part = part0 + k;
      out.items.push_back(p);
    }
    out.n_parts += k;
    out.merges.push_back(PrefillMerge{it.entry, it.kvh, it.q0, it.nq, part0, k, 0, 0});
  }
  // Most tiles first; then, among the first resident workgroups, the second half in
  // reverse: workgroups w and w + kPrefillResident / 2 are placed on one CU, which so
  // gets one long and one short item (the causal items of a first chunk hold 1 to 64
  // tiles) instead of two long or two short ones.
  order_prefill_items(out.items.data(), out.items.size());
  const size_t half = kPrefillResident / 2, window = std::min<size_t>(out.items.size(), kPrefillResident);
  if (window > half) std::reverse(out.items.begin() + half, out.items.begin() + window);
}

}  // namespace hxf
