// Launch order of a step's attention items (host code).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

namespace hvd {

constexpr int kXcds = 8;

// One item: KV chunk `chunk` of unit `unit` (a row group of the (sequence, kv
// head) `stream`), `keys` positions long.
struct AttnPiece {
  int stream, unit, chunk, keys;
};

// The pieces in unit order, but for streams of several units (row groups that read
// the same chunks): there the units' pieces of one chunk go kXcds positions apart,
// next to each other in dispatch order -- the same XCD at nearly the same time,
// so that a chunk comes from HBM once and from that XCD's L2 for the others.
// Chunks in runs of kXcds: run position j of unit r at run base + kXcds r + j, a
// no-op piece (unit -1) where a unit has fewer chunks.  Pieces in unit order.
inline std::vector<AttnPiece> attn_interleave(const std::vector<AttnPiece>& in) {
  std::vector<AttnPiece> out;
  out.reserve(in.size() + in.size() / 4);
  std::vector<size_t> unit;  // first piece of each unit of the stream, and the end
  for (size_t i0 = 0, i1; i0 < in.size(); i0 = i1) {
    unit.clear();
    for (i1 = i0; i1 < in.size() && in[i1].stream == in[i0].stream; ++i1)
      if (i1 == i0 || in[i1].unit != in[i1 - 1].unit) unit.push_back(i1);
    unit.push_back(i1);
    const size_t n = unit.size() - 1;
    if (n == 1) {
      out.insert(out.end(), in.begin() + i0, in.begin() + i1);
      continue;
    }
    size_t most = 0;
    for (size_t r = 0; r < n; ++r) most = std::max(most, unit[r + 1] - unit[r]);
    for (size_t c0 = 0; c0 < most; c0 += kXcds)
      for (size_t r = 0; r < n; ++r)
        for (size_t c = c0; c < std::min(most, c0 + kXcds); ++c)
          out.push_back(c < unit[r + 1] - unit[r] ? in[unit[r] + c] : AttnPiece{-1, -1, 0, 0});
  }
  return out;
}

// Whether a launch of these pieces on `cus` compute units, one per unit at a time, ends
// sooner with the longest first.  In any other order every round may hold one of
// the longest pieces; longest first it takes its keys shared evenly, or the rounds
// of the longest ones alone (a round of a sixteenth of the CUs is not counted: its
// few workgroups have the memory to themselves).  Where that saves less than a tenth,
// or the pieces are so short that their fixed cost decides, the host pays more for
// the order (a median of 14 us per step) than the launch gains.
// Measured over 275 batches (2 to 32 sequences, 100 to 16384 keys, five head
// layouts, 4 layers): where the rounds are equal steps by length took 17 us longer
// and the attention as long; where the rule holds the attention was up to 50%
// faster (two 65-row drafts at 16384: 487 -> 323 us).  All steps together took 1% less
// than ordered wherever there are more items than CUs.
inline bool attn_order_pays(const std::vector<AttnPiece>& pieces, int cus) {
  int longest = 0;
  for (const AttnPiece& p : pieces) longest = std::max(longest, p.keys);
  if (longest < 128) return false;
  int64_t total = 0, n_longest = 0;
  for (const AttnPiece& p : pieces) {
    total += p.keys;
    n_longest += p.keys == longest;
  }
  auto rounds = [&](int64_t n) { return (n + cus - 1) / cus * longest; };
  const int64_t alone = std::max<int64_t>(longest, rounds(std::max<int64_t>(0, n_longest - cus / 16)));
  return 10 * rounds((int64_t)pieces.size()) >= 11 * std::max(alone, total / cus);
}

// Stable sort of `order` (indexes) by descending key: least significant byte
// first, as many passes as the largest key has bytes.
template <class Key>
inline void attn_sort_desc(std::vector<int>& order, const Key& key) {
  int64_t most = 0;
  for (int i : order) most = std::max<int64_t>(most, key(i));
  std::vector<int> from(order.size());
  for (int shift = 0; most >> shift > 0; shift += 8) {
    size_t at[257] = {};
    order.swap(from);
    for (int i : from) ++at[256 - ((key(i) >> shift) & 255)];
    for (int b = 1; b < 257; ++b) at[b] += at[b - 1];
    for (int i : from) order[at[255 - ((key(i) >> shift) & 255)]++] = i;
  }
}

// The items as kXcds interleaved queues: workgroup i runs on XCD i % kXcds
// (round-robin dispatch), so position i belongs to queue i % kXcds.  The items
// of one (stream, chunk) read the same keys and go to one queue; these bundles
// are dealt to the least loaded queue, largest first (ties: in order), and a
// queue runs its longest items first (ties: by stream, chunk, unit).  Bundles too
// few or too uneven to balance the queues are dealt item by item instead.
// Shorter queues are filled with no-op pieces (unit -1), never more of them
// than items; queues of too different lengths fall back to plain length order.
// The pieces come in unit order: streams and units ascending, each unit's
// chunks from 0 up.  Linear time, since the GPU waits for a step's plan (by
// comparison sorts 3900 items took 362 us, here 74; 512 25 and 11).
inline std::vector<AttnPiece> attn_order(const std::vector<AttnPiece>& in) {
  const size_t n = in.size();
  // by stream, chunk, unit
  std::vector<AttnPiece> pieces(n);
  std::vector<size_t> at;
  for (size_t i0 = 0, i1; i0 < n; i0 = i1) {
    at.assign(1, i0);
    for (i1 = i0; i1 < n && in[i1].stream == in[i0].stream; ++i1) {
      if ((size_t)in[i1].chunk + 2 > at.size()) at.resize(in[i1].chunk + 2, 0);
      ++at[in[i1].chunk + 1];
    }
    for (size_t c = 1; c < at.size(); ++c) at[c] += at[c - 1];
    for (size_t i = i0; i < i1; ++i) pieces[at[in[i].chunk]++] = in[i];
  }
  std::vector<int64_t> keys;        // of each bundle
  std::vector<int> first, order, queue_of(n);
  auto deal = [&](bool whole) {
    keys.clear();
    first.clear();
    for (size_t i = 0; i < n; ++i) {
      if (!whole || i == 0 || pieces[i].stream != pieces[i - 1].stream || pieces[i].chunk != pieces[i - 1].chunk) {
        keys.push_back(0);
        first.push_back((int)i);
      }
      keys.back() += pieces[i].keys;
    }
    order.resize(keys.size());
    for (size_t b = 0; b < order.size(); ++b) order[b] = (int)b;
    attn_sort_desc(order, [&](int b) { return keys[b]; });
    first.push_back((int)n);
    int64_t load[kXcds], total = 0;  // load * kXcds + queue: the least is the first of the least loaded
    for (int x = 0; x < kXcds; ++x) load[x] = x;
    for (int b : order) {
      int64_t least = load[0];
      for (int x = 1; x < kXcds; ++x) least = std::min(least, load[x]);
      const int x = (int)(least % kXcds);
      load[x] += keys[b] * kXcds;
      total += keys[b];
      for (int i = first[b]; i < first[b + 1]; ++i) queue_of[i] = x;
    }
    return *std::max_element(load, load + kXcds) / kXcds * kXcds <= total + total / 8;
  };
  if (!deal(true) && keys.size() < n) deal(false);
  order.resize(n);
  for (size_t i = 0; i < n; ++i) order[i] = (int)i;
  attn_sort_desc(order, [&](int i) { return pieces[i].keys; });
  size_t len[kXcds] = {};
  for (int x : queue_of) ++len[x];
  const size_t longest = *std::max_element(len, len + kXcds);
  std::vector<AttnPiece> out;
  if (longest * kXcds > 2 * n) {
    for (int i : order) out.push_back(pieces[i]);
    return out;
  }
  out.assign(longest * kXcds, AttnPiece{-1, -1, 0, 0});
  size_t pos[kXcds];
  for (int x = 0; x < kXcds; ++x) pos[x] = x;
  for (int i : order) {
    out[pos[queue_of[i]]] = pieces[i];
    pos[queue_of[i]] += kXcds;
  }
  while (!out.empty() && out.back().unit < 0) out.pop_back();
  return out;
}

}  // namespace hvd
