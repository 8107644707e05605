// Work plan of the GEMMs of 33 to 128 verify rows (host code): columns per
// workgroup, K splits and row blocks of gemm_mid.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace hvd {

constexpr int kMidMinMT = 3, kMidMaxMT = 8;  // row tiles gemm_mid takes, at least and per row block
constexpr int kMidMinDim = 4096;             // GEMMs of fewer columns or a shorter K do not use it
constexpr int kGemmSplitTarget = 256;        // workgroups a K split aims for (one per CU)
constexpr int kGemmLongK = 256;              // K steps above which a K split pays for its reduction
constexpr int kGemmCounters = 16384;         // split-K arrival counters (output blocks of one launch)

// strips of 16 columns per workgroup (4 or 8), K splits, row blocks and their row tiles
struct MidPlan {
  int strips, splits, mblocks, mt_block;
};

// Three row tiles or more: gemm_mid, whose waves share the activations.
// Measured per verify step against gemm_skinny (context 2048), 8 layers of
// the 8B shape: 34 rows 1343 -> 1257 us, 51 1533 -> 1423, 65 1721 -> 1563,
// 96 2009 -> 1665, 128 2239 -> 1866; 4 layers of the 32B widths: 41 rows
// 1605 -> 1296 us, 128 2767 -> 1842.  At two row tiles it is no faster (8B,
// 17 rows: 3.95 against 3.94 ms).  Small shapes leave a workgroup a short K range
// or many splits, and its fixed cost decides: all GEMMs of width 2048 through
// gemm_mid 650 -> 642 us at 41 rows, 711 -> 718 at 64 and 836 -> 967 at 128
// (8 layers), of width 512 380 -> 392, 411 -> 415 and 427 -> 554.
// Its activation offsets are 32-bit: operands of 2 GiB or more (75000 rows of K
// 14336, where N is no multiple of 128 and the tiled kernel cannot run) stay
// with gemm_skinny.
inline bool mid_takes(int mtiles, int N, int K) {
  return mtiles >= kMidMinMT && K >= kMidMinDim && N >= kMidMinDim && (int64_t)mtiles * (K / 32) * 1024 <= INT32_MAX;
}

// 128 columns per workgroup where those fill the CUs, and for long K (fewer
// activation bytes per weight byte); else 64, whose K splits have half
// the partial tile to publish and sum (72 rows of the 8B shape: O with
// 64 columns and 4 splits against 128 and 8 2.6 us per layer less, QKV
// with 64 and 2 against 128 and 5 2.7 us less; down with 64 and 4 against
// 128 and 8 0.6 us more).  No split that needs a second round of the CUs.
// A split's partial tiles take as many bytes with either width: where part_bytes
// cuts the splits of 128 columns, 64 columns and as many splits run twice the
// workgroups (hvd_verify_noalloc with its 8 MiB, 128 rows: down of the 8B shape on
// 256 against 128, the step of 4 layers 1122 -> 1024 us; 2 layers of the 32B
// widths 1243 -> 1109).
// wide: whether 128 columns are allowed at up to four row tiles; force: {strips,
// splits} of a tuning override (strips 0: none), rounded to what gemm_mid has.
inline MidPlan mid_plan(int mtiles, int NT, int KT, int min_blocks, bool wide, size_t part_bytes, const int* force) {
  MidPlan p;
  p.mblocks = (mtiles + kMidMaxMT - 1) / kMidMaxMT;
  p.mt_block = (mtiles + p.mblocks - 1) / p.mblocks;
  const bool can8 = NT % 8 == 0 && (wide || p.mt_block > 4);
  auto units = [&](int strips) { return NT / strips * p.mblocks; };
  auto filled = [&](int u) { return u * std::max(1, kGemmSplitTarget / u); };
  auto splits = [&](int strips) {
    const int u = units(strips);
    int s = std::max(1, std::min({force[0] ? force[1] : kGemmSplitTarget / u, KT / 8, 16}));
    while (s > 1 && (size_t)u * s * p.mt_block * 16 * strips * 16 * 4 > part_bytes) --s;
    return u > kGemmCounters ? 1 : s;
  };
  const int u4 = units(4), u8 = units(8);
  p.strips = can8 && (u8 >= min_blocks || KT >= kGemmLongK || 4 * filled(u4) < 3 * filled(u8)) ? 8 : 4;
  if (force[0]) p.strips = force[0] >= 8 && NT % 8 == 0 ? 8 : 4;
  p.splits = splits(p.strips);
  if (!force[0] && p.strips == 8 && p.splits < kGemmSplitTarget / u8 && u4 * splits(4) > u8 * p.splits) {
    p.strips = 4;
    p.splits = splits(4);
  }
  return p;
}

}  // namespace hvd
