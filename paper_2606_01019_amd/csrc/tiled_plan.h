// Work plan of the large-batch GEMMs (host code): which tile, how many
// workgroups, and which tiles are shared by several workgroups along K.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#ifdef __HIPCC__
#define HVD_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define HVD_HOST_DEVICE inline
#endif

namespace hvd {

constexpr int kTiles = 5;
constexpr int kTileBM[kTiles] = {128, 128, 256, 256, 128};
constexpr int kTileBN[kTiles] = {128, 256, 256, 256, 256};

// n_wg workgroups.  The last n_shared tiles of the grid are shared: their K
// steps, taken as one list, are dealt to the first n_sk workgroups in equal
// contiguous runs (the published "stream-K" decomposition); the other tiles go whole to the workgroups in turn.
// n_shared < n_sk <= n_wg, so that a run spans at most two tiles.
struct TiledPlan {
  int tile = 0, n_wg = 0, n_shared = 0, n_sk = 0;
};

// The shared K steps, counted through the shared tiles in order (tile t holds
// steps t KT .. t KT + KT - 1), and the runs they are dealt out in: worker w
// has steps [lo(w), lo(w + 1)).  With as many workers for every tile (parts > 0)
// each tile's steps are cut alike and worker w's part goes to partial slot w.
// Otherwise a run may span two tiles, and its part of shared tile t goes to slot
// w + t (distinct, since runs are contiguous, and consecutive per tile).
struct SharedRuns {
  int KT, q, r, n_shared, n_sk, parts;
  HVD_HOST_DEVICE SharedRuns(int n_shared_, int KT_, int n_sk_)
      : KT(KT_), q(n_sk_ ? n_shared_ * KT_ / n_sk_ : 0), r(n_sk_ ? n_shared_ * KT_ % n_sk_ : 0), n_shared(n_shared_),
        n_sk(n_sk_), parts(n_sk_ && n_sk_ % n_shared_ == 0 ? n_sk_ / n_shared_ : 0) {}
  HVD_HOST_DEVICE int lo(int w) const {
    return parts ? w / parts * KT + w % parts * KT / parts : w * q + (w < r ? w : r);
  }
  // the worker whose run holds a step
  HVD_HOST_DEVICE int holder(int step) const {
    if (parts) return step / KT * parts + ((step % KT + 1) * parts - 1) / KT;
    const int cut = r * (q + 1);
    return step < cut ? step / (q + 1) : r + (step - cut) / q;
  }
  // worker w's partial slot of shared tile t is slot0(w) + t
  HVD_HOST_DEVICE int slot0(int w) const { return parts ? w - w / parts : w; }
  // worker of the l-th workgroup in XCD order: with a uniform split, the same
  // K range of neighbouring tiles goes to neighbours, which share its
  // operands in their L2 (328 rows x 5120 columns, K 27648: 228 -> 218 us)
  HVD_HOST_DEVICE int worker(int l) const {
    return parts ? l % n_shared * parts + l / n_shared : l;
  }
};

// What the kernels assume of a plan for T tiles of KT K steps: every shared K
// step has a workgroup, a run spans at most two tiles, and no run covers a whole
// tile -- gemm_tiled takes a part that does for a whole tile of its own and
// publishes nothing, and tiled_finish would sum the slot it left unwritten.
inline bool tiled_plan_ok(const TiledPlan& p, int T, int KT) {
  const int64_t steps = (int64_t)p.n_shared * KT;
  if (p.n_wg < 1 || p.n_shared < 0 || p.n_shared > T || p.n_sk > p.n_wg || (p.n_shared > 0) != (p.n_sk > 0)) return false;
  if (!p.n_shared) return true;
  return steps >= p.n_sk && steps <= INT32_MAX && (steps + p.n_sk - 1) / p.n_sk < KT;
}

// Bytes of partial slots the plan needs.  An even split needs one per worker:
// 8 MiB (hvd_verify_noalloc) then hold a two-way split of 256 rows x 4096 columns,
// 64 workgroups instead of 32 (4 layers of the 8B widths, 130 rows: 2.72 -> 1.97 ms).
inline size_t tiled_partial_bytes(const TiledPlan& p) {
  if (!p.n_shared) return 0;
  return (size_t)(p.n_sk + (p.n_sk % p.n_shared ? p.n_shared : 0)) * kTileBM[p.tile] * kTileBN[p.tile] * 4;
}

// `splits`-way K split of every tile (1: whole tiles), for tuning overrides.
inline TiledPlan tiled_plan_forced(int tile, int splits, int mtiles, int N, int KT, size_t part_bytes) {
  const int T = (mtiles * 16 + kTileBM[tile] - 1) / kTileBM[tile] * (N / kTileBN[tile]);
  for (splits = std::min(splits, KT); splits > 1; --splits) {
    const TiledPlan p{tile, T * splits, T, T * splits};
    if (tiled_partial_bytes(p) <= part_bytes) return p;
  }
  return TiledPlan{tile, T, 0, 0};
}

// The plan with the least estimated time.  The estimate (microseconds) is
// fitted to a sweep of every plan below over 144 - 2048 rows of the 8B and
// 32B shapes' GEMMs; it orders them as measured within about 5%:
//  * a K step of 32 on a 128 x 256 tile (8 waves) takes 0.9 on the hi + lo
//    pair and 0.53 single-pass while all CUs are busy (0.66 and 0.39 on a
//    quarter of them: the clock falls under load), a 256 x 256 tile's 1.6 and
//    0.9: fewer operand bytes per MFMA, so it wins wherever its rounds fill
//    the CUs (512 rows x 28672: 218 against 239);
//  * the 4-wave 128 x 256 tile runs two workgroups per CU single-pass, so its
//    epilogues overlap (LM head, 853 rows: 948 against 1002 with 256 x 256);
//  * runs that do not cut every tile alike read their operands at other K
//    offsets than their neighbours: 15% per step;
//  * shared tiles cost a second launch and its reads of the partials.
// part_bytes bounds the partial tiles.
inline TiledPlan tiled_plan(int mtiles, int N, int KT, bool single, int cus, size_t part_bytes) {
  constexpr int kMinRun = 8;       // K steps below which a shared run does not pay
  constexpr double kLaunch = 5.0, kFinish = 5.0, kPartRate = 4.0e6;  // partial bytes per microsecond
  TiledPlan best;
  double best_us = 1e30;
  auto consider = [&](const TiledPlan& p, double us) {
    if (tiled_partial_bytes(p) > part_bytes || us >= best_us) return;
    best = p;
    best_us = us;
  };
  auto tiles_of = [&](int t) { return (mtiles * 16 + kTileBM[t] - 1) / kTileBM[t] * (N / kTileBN[t]); };
  if (N % 256 != 0) {  // 128 x 128 tiles, two workgroups per CU
    const int T = tiles_of(0);
    const int s = T >= 2 * cus ? 1 : std::max(1, std::min({4, 2 * cus / T, KT / 32}));
    return tiled_plan_forced(0, s, mtiles, N, KT, part_bytes);
  }
  if (single) {
    const int T = tiles_of(1), rest = T % (2 * cus);
    consider(TiledPlan{1, T, 0, 0}, kLaunch + KT * 1.05 * (T / (2 * cus) + (rest > cus ? 1.0 : rest ? 0.6 : 0.0)));
  }
  for (int t : {4, 2}) {
    const int T = tiles_of(t), rest = T % cus;
    const double step = t == 4 ? (single ? 0.53 : 0.9) : (single ? 0.9 : 1.6), epi = t == 4 ? 5.0 : 8.0;
    // steps of one workgroup, as a time, when `busy` of them run at once
    auto run = [&](double steps, int busy) { return steps * step * (0.73 + 0.27 * std::min(busy, cus) / cus); };
    const double whole = T / cus * (run(KT, cus) + epi);  // full rounds
    consider(TiledPlan{t, T, 0, 0}, kLaunch + whole + (rest ? run(KT, rest) + epi : 0.0));
    if (!rest) continue;
    const int n_wg = T < cus ? 0 : cus;  // (0: as many as share)
    auto shared = [&](int n_sk, double factor) {
      const TiledPlan p{t, std::max(n_wg, n_sk), rest, n_sk};
      if (!tiled_plan_ok(p, T, KT)) return;
      const int steps = (int)(((int64_t)rest * KT + n_sk - 1) / n_sk);
      consider(p, kLaunch + whole + run(steps, n_sk) * factor + kFinish + (double)(n_sk + rest) * kTileBM[t] * kTileBN[t] * 4 / kPartRate + epi);
    };
    for (int s = 2; s <= 16 && rest * s <= cus && KT / s >= kMinRun; ++s) shared(rest * s, 1.0);
    const int n_sk = (int)std::min<int64_t>(cus, (int64_t)rest * KT / kMinRun);
    if (n_sk > rest && n_sk % rest) shared(n_sk, 1.15);
  }
  return best;
}

}  // namespace hvd
