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

// The items as kXcds interleaved queues: workgroup i runs on XCD i % kXcds
// (round-robin dispatch), so position i belongs to queue i % kXcds.  The items
// of one (stream, chunk) read the same keys and go to one queue; these bundles
// are dealt to the least loaded queue, largest first (ties: in order), and a
// queue runs its longest items first (ties: by stream, chunk, unit).  Bundles too
// few or too uneven to balance the queues are dealt item by item instead.
// Shorter queues are filled with no-op pieces (unit -1), never more of them
// than items; queues of too different lengths fall back to plain length order.
inline std::vector<AttnPiece> attn_order(std::vector<AttnPiece> pieces) {
  struct Bundle { int64_t keys; size_t first, n; };
  auto before = [](const AttnPiece& a, const AttnPiece& b) {
    if (a.stream != b.stream) return a.stream < b.stream;
    if (a.chunk != b.chunk) return a.chunk < b.chunk;
    return a.unit < b.unit;
  };
  auto longer = [&](const AttnPiece& a, const AttnPiece& b) { return a.keys != b.keys ? a.keys > b.keys : before(a, b); };
  std::vector<AttnPiece> queue[kXcds];
  auto deal = [&](bool whole) {
    std::vector<Bundle> bundles;
    for (size_t i = 0; i < pieces.size(); ++i) {
      const AttnPiece& a = pieces[i];
      if (!whole || i == 0 || a.stream != pieces[i - 1].stream || a.chunk != pieces[i - 1].chunk)
        bundles.push_back({0, i, 0});
      bundles.back().keys += a.keys;
      bundles.back().n += 1;
    }
    std::stable_sort(bundles.begin(), bundles.end(), [](const Bundle& a, const Bundle& b) { return a.keys > b.keys; });
    int64_t load[kXcds] = {}, total = 0;
    for (auto& q : queue) q.clear();
    for (const Bundle& b : bundles) {
      const int x = (int)(std::min_element(load, load + kXcds) - load);
      load[x] += b.keys;
      total += b.keys;
      queue[x].insert(queue[x].end(), pieces.begin() + b.first, pieces.begin() + b.first + b.n);
    }
    return *std::max_element(load, load + kXcds) * kXcds <= total + total / 8;
  };
  std::sort(pieces.begin(), pieces.end(), before);
  if (!deal(true)) deal(false);
  size_t longest = 0;
  for (auto& q : queue) {
    std::sort(q.begin(), q.end(), longer);
    longest = std::max(longest, q.size());
  }
  std::vector<AttnPiece> out;
  if (longest * kXcds > 2 * pieces.size()) {
    std::sort(pieces.begin(), pieces.end(), longer);
    return pieces;
  }
  for (size_t i = 0; i < longest; ++i)
    for (auto& q : queue) out.push_back(i < q.size() ? q[i] : AttnPiece{-1, -1, 0, 0});
  while (!out.empty() && out.back().unit < 0) out.pop_back();
  return out;
}

}  // namespace hvd
