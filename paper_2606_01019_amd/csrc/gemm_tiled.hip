// Large-batch GEMMs of the verify forward (gfx950, MFMA 32x32x16 f16): many
// verify rows at once (batched sequences, long drafts) and prefill chunks,
// where the weight-streaming kernel would re-read the weights per 64 rows.
//
// Y[m, n] = sum_k A[m, k] W[n, k] over the same packed operands as the
// streaming kernel: 1 KB fragments of 16 rows (or weight columns) x 32 K.
// A workgroup of WY x WX waves owns a BM x BN tile (BM = 32 WM WY, BN =
// 32 WN WX) and walks its K range in 32-wide steps: every step's A and W
// fragments are copied from global memory straight into a ring of ST LDS
// slots (global_load_lds: no registers, ST - 1 steps in flight ahead of the
// MFMAs), and each wave multiplies its 32WM x 32WN sub-tile with WM x WN
// MFMA tiles of 32 x 32.
// The 256 x 256 tile (8 waves) needs about 32 bytes of operand per clock and
// CU at full MFMA rate; 128-row tiles (4 waves) serve smaller batches.
// HI_LO chooses the activation precision: the fp16 hi + lo pair (two MFMAs
// per tile, ~22 bits) or the hi part alone (one MFMA, 11 bits).
//
// Work: every workgroup takes whole tiles in turn; tiles that would leave
// CUs idle are shared, their K steps dealt out in equal runs (tiled_plan.h).
// Workgroups are numbered so that each XCD receives neighbouring tiles, the
// row blocks of a column block adjacent: the weight tile is fetched from HBM
// once into that XCD's L2 and re-read from there by the other row blocks.
// Shared tiles write fp32 partial tiles, which tiled_finish sums in K order.
//
// MFMA 32x32 output element of register r: row 8*(r/4) + 4*(lane/32) + r%4,
// column lane%32.  The epilogue turns it through LDS (epi_block).
#include "common.h"
#include "kernels.h"

#include <type_traits>

namespace hvd {

typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ f32x16 mfma32_f16(const u32x4& a, const u32x4& b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                0, 0);
}

// Workgroup id -> position in a list of `total` workgroups whose neighbours
// share an XCD: XCD x (= id % 8 under the round-robin dispatch) gets the run
// [start_x, start_x + n_x).
__device__ __forceinline__ int xcd_run(int id, int total) {
  const int x = id & 7, local = id >> 3;
  const int q = total >> 3, rem = total & 7;
  return x * q + min(x, rem) + local;
}

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// ---- Epilogues, on blocks of 32 rows x 64 columns of one wave.
//
// The MFMA layout holds a column per lane, where every output wants several
// columns (or, for V, rows) of one element group in one store: the block goes
// through the wave's own LDS region and comes back as octets of 8 columns of
// one row, so that the stores are 16 bytes per lane.  (Stored from the MFMA
// layout, 2 bytes per lane, the epilogue of a 128 x 256 tile took about 24 us
// of the 107 us of a 4096-deep product on the hi + lo pair.)
constexpr int kEpiStride = 72;                    // floats per row: rows 4 apart land 32 banks apart
constexpr int kEpiBytes = 32 * kEpiStride * 4;    // LDS region of one wave

// Residual inputs of a block, requested before the previous block's stores: a
// load issued after a store waits for that store before its value can be used.
template <int EPI>
struct EpiX {
  static constexpr bool ON = EPI == EPI_RESID;
  float4 x[ON ? 4 : 1][2], gain[2];
};

template <int EPI>
__device__ __forceinline__ void epi_load_x(const GemmArgs& a, int row0, int col0, EpiX<EPI>& e) {
  if constexpr (EPI == EPI_RESID) {
    const int lane = threadIdx.x & 63;
    const int C = col0 + (lane & 7) * 8;
    e.gain[0] = *(const float4*)(a.gain_next + C);
    e.gain[1] = *(const float4*)(a.gain_next + C + 4);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int R = min(row0 + (lane >> 3) + 8 * it, a.M - 1);
      const float4* xp = (const float4*)(a.X + (size_t)R * a.D + C);
      e.x[it][0] = xp[0];
      e.x[it][1] = xp[1];
    }
  }
}

// c0, c1: the two 32 x 32 accumulators of the block at (row0, col0); lds: the
// wave's region.  inv_rms: per-row inverse RMS (GEMMs of normalised inputs).
template <int EPI>
__device__ __forceinline__ void epi_block(const GemmArgs& a, const f32x16& c0, const f32x16& c1, int row0, int col0,
                                          const float* __restrict__ inv_rms, const EpiX<EPI>& ex, float* lds) {
  const int lane = threadIdx.x & 63;
  const int lhi = lane >> 5, lc = lane & 31;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float* p = lds + (8 * (r >> 2) + 4 * lhi + (r & 3)) * kEpiStride + lc;
    p[0] = c0[r];
    p[32] = c1[r];
  }
  // (one wave's LDS accesses execute in order)
  __builtin_amdgcn_wave_barrier();
  auto oct = [&](int row, int c, float (&v)[8]) __attribute__((always_inline)) {
    const float4 x = *(const float4*)(lds + row * kEpiStride + c), y = *(const float4*)(lds + row * kEpiStride + c + 4);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
  };
  if constexpr (EPI == EPI_RESID) {
    const int o = lane & 7, C = col0 + o * 8;
    const float gn[8] = {ex.gain[0].x, ex.gain[0].y, ex.gain[0].z, ex.gain[0].w,
                         ex.gain[1].x, ex.gain[1].y, ex.gain[1].z, ex.gain[1].w};
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int row = (lane >> 3) + 8 * it, R = row0 + row;
      float v[8];
      oct(row, o * 8, v);
      const float4 xa = ex.x[it][0], xb = ex.x[it][1];
      v[0] += xa.x; v[1] += xa.y; v[2] += xa.z; v[3] += xa.w;
      v[4] += xb.x; v[5] += xb.y; v[6] += xb.z; v[7] += xb.w;
      float sq = 0.f, n[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        sq += v[i] * v[i];
        n[i] = v[i] * gn[i];
      }
      sq += __shfl_xor(sq, 1);  // the strip's other octet
      if (R < a.M) {
        float4* xp = (float4*)(a.X + (size_t)R * a.D + C);
        xp[0] = float4{v[0], v[1], v[2], v[3]};
        xp[1] = float4{v[4], v[5], v[6], v[7]};
        uint4 hi, lo;
        split8(n, hi, lo);
        const size_t off = afrag_off(R, C, a.MTtot);
        *(uint4*)(a.Nhi + off) = hi;
        *(uint4*)(a.Nlo + off) = lo;
        if ((o & 1) == 0) a.ss_out[(size_t)R * (a.D >> 4) + (C >> 4)] = sq;
      }
    }
  } else if constexpr (EPI == EPI_SILU) {
    // a 32-column tile is one (gate strip, up strip) pair
    const int o = lane & 3, c = 32 * (o >> 1) + 8 * (o & 1), F = (col0 >> 1) + o * 8;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const int row = (lane >> 2) + 16 * it, R = row0 + row;
      const float ir = inv_rms[min(R, a.M - 1)];
      float g[8], u[8];
      oct(row, c, g);
      oct(row, c + 16, u);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float v = g[i] * ir;
        u[i] = v / (1.f + __expf(-v)) * (u[i] * ir);
      }
      if (R < a.M) {
        uint4 hi, lo;
        split8(u, hi, lo);
        const size_t off = afrag_off(R, F, a.MTtot);
        *(uint4*)(a.act_hi + off) = hi;
        *(uint4*)(a.act_lo + off) = lo;
      }
    }
  } else if constexpr (EPI == EPI_QKV) {
    // heads are 64 or 128 columns wide: the block lies within q, k or v
    if (col0 < a.q_cols + a.kv_cols) {
      const int o = lane & 7, C = col0 + o * 8;
      const int base = C < a.q_cols ? 0 : a.q_cols;
      const int hg = (C - base) / a.dh, dp = (C - base) % a.dh;
      RowMeta rm[4];
      float ir[4];
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int R = min(row0 + (lane >> 3) + 8 * it, a.M - 1);
        rm[it] = a.rows[R];
        ir[it] = inv_rms[R];
      }
      float4 cs[4][2];  // 4 rotary (cos, sin) pairs
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const float4* rp = (const float4*)(a.rope + (size_t)rm[it].pos * (a.dh >> 1) + (dp >> 1));
        cs[it][0] = rp[0];
        cs[it][1] = rp[1];
      }
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int row = (lane >> 3) + 8 * it, R = row0 + row;
        float v[8];
        oct(row, o * 8, v);
        const float4 ca = cs[it][0], cb = cs[it][1];
        const float cc[4] = {ca.x, ca.z, cb.x, cb.z}, sn[4] = {ca.y, ca.w, cb.y, cb.w};
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v0 = v[2 * i] * ir[it], v1 = v[2 * i + 1] * ir[it];
          w[i] = pack_h2(v0 * cc[i] - v1 * sn[i], v1 * cc[i] + v0 * sn[i]);
        }
        if (R < a.M) {
          _Float16* dst = C < a.q_cols ? a.Q + (size_t)R * a.q_cols + C
                                       : a.kv + (size_t)(rm[it].kvs / kPage) * a.page_stride +
                                             ((size_t)hg * kPage + (rm[it].kvs & (kPage - 1))) * a.dh + dp;
          *(uint4*)dst = uint4{w[0], w[1], w[2], w[3]};
        }
      }
    } else {
      // V is [dim][16 positions] in a page: eight rows that hold eight
      // consecutive positions from a multiple of 8 are one 16-byte store
      const int R = row0 + lc;
      const int kvsl = R < a.M ? a.rows[R].kvs : -1;
      const float irl = inv_rms[min(R, a.M - 1)];
      const int first = __shfl(kvsl, lc & 24);
      const uint32_t whole = (uint32_t)__builtin_amdgcn_ballot_w64(kvsl >= 0 && (first & 7) == 0 && kvsl == first + (lc & 7));
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int grp = 2 * (it >> 1) + (lane & 1), col = 32 * (it & 1) + (lane >> 1);
        const int cv = col0 + col - a.q_cols - a.kv_cols;
        _Float16* vcol = a.kv + (size_t)a.Hkv * kPage * a.dh + (size_t)cv * kPage;  // (head * dh + dim) * 16
        float v[8];
        int slot[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[e] = lds[(8 * grp + e) * kEpiStride + col] * __shfl(irl, 8 * grp + e);
          slot[e] = __shfl(kvsl, 8 * grp + e);
        }
        if (((whole >> (8 * grp)) & 0xffu) == 0xffu) {
          *(uint4*)(vcol + (size_t)(slot[0] / kPage) * a.page_stride + (slot[0] & (kPage - 1))) =
              uint4{pack_h2(v[0], v[1]), pack_h2(v[2], v[3]), pack_h2(v[4], v[5]), pack_h2(v[6], v[7])};
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (slot[e] >= 0) vcol[(size_t)(slot[e] / kPage) * a.page_stride + (slot[e] & (kPage - 1))] = (_Float16)v[e];
        }
      }
    }
  } else {  // EPI_LM: logits, and per row the max / lowest argmax over the 64 columns
    const int o = lane & 7, C = col0 + o * 8;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int row = (lane >> 3) + 8 * it, R = row0 + row;
      const float ir = inv_rms[min(R, a.M - 1)];
      float v[8];
      oct(row, o * 8, v);
      float best = -INFINITY;
      int bidx = 0x7fffffff;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        v[i] *= ir;
        if (v[i] > best) {  // columns ascend: ties keep the lower one
          best = v[i];
          bidx = C + i;
        }
      }
#pragma unroll
      for (int s = 1; s < 8; s <<= 1) {
        const float ov = __shfl_xor(best, s);
        const int oi = __shfl_xor(bidx, s);
        if (ov > best || (ov == best && oi < bidx)) {
          best = ov;
          bidx = oi;
        }
      }
      if (R < a.M) {
        if (a.logits) store_logits8(a.logits + (size_t)R * a.vocab + C, v);
        if (o == 0) {
          a.part_val[(size_t)R * a.n_part + (col0 >> 6)] = best;
          a.part_idx[(size_t)R * a.n_part + (col0 >> 6)] = bidx;
        }
      }
    }
  }
  __builtin_amdgcn_wave_barrier();
}

// 128 x 128 wave tiles (256 accumulators) run one wave per SIMD
constexpr int tiled_occupancy(int WM, int WN) { return WM * WN >= 16 ? 1 : 2; }

template <int WY, int WX, int WM, int WN, int EPI, bool HI_LO>
__global__ __launch_bounds__(64 * WY * WX, tiled_occupancy(WM, WN)) void gemm_tiled(
    GemmArgs a, const float* __restrict__ inv_rms, int RB, int CB, int n_shared, int n_sk) {
  constexpr int NW = WY * WX;
  constexpr int BM = 32 * WM * WY, BN = 32 * WN * WX;
  constexpr int AF = BM / 16;              // A fragments per K step
  constexpr int NA = HI_LO ? 2 * AF : AF;  // with the lo part
  constexpr int WF = BN / 16;              // weight fragments per K step
  constexpr int NF = NA + WF;
  constexpr int LPT = NF / NW;  // 16-byte loads per thread per K step (NF*64 / (64*NW))
  static_assert(NF % NW == 0, "fragments per step");
  // ring depth: two workgroups per CU for the small tiles, else one
  constexpr int LDS_BUDGET = (NW == 4 && WM * WN < 16) ? 76 * 1024 : 150 * 1024;
  constexpr int ST0 = LDS_BUDGET / (NF * 1024);
  constexpr int ST = ST0 < 3 ? 3 : (ST0 > 6 ? 6 : ST0);
  __shared__ u32x4 sbuf[ST][NF][64];
  static_assert(NW * kEpiBytes <= (int)sizeof(sbuf), "the epilogue's regions fit the ring");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wy = wave / WX, wx = wave % WX;
  // operand fragment of 32 rows (or columns) starting at fragment f0, K
  // sub-step s (16 of the 32): lane l takes row l%32, K 16s + 8(l/32)..+8
  const int fl = (lane & 15) + 16 * (lane >> 5);  // lane within the fragment, s = 0
  const int fo = (lane >> 4) & 1;                 // second fragment for lanes 16-31 / 48-63

  // This workgroup's work: first its share of the n_shared tiles (the
  // last ones of the grid of RB x CB), whose K steps are dealt to n_sk
  // workgroups in equal contiguous runs; then every gridDim.x-th whole tile.
  const int T = RB * CB, n_whole = T - n_shared;
  const int KT = a.KT;
  const SharedRuns runs(n_shared, KT, n_sk);
  int lo = 0, hi = 0, slot0 = 0;  // this workgroup's run of the shared K steps, and its partial slots
  if ((int)blockIdx.x < n_sk) {
    const int w = runs.worker(xcd_run(blockIdx.x, n_sk));
    lo = runs.lo(w);
    hi = runs.lo(w + 1);
    slot0 = runs.slot0(w);
  }
  int whole = xcd_run(blockIdx.x, gridDim.x);
  bool first = true;

  for (;;) {
  int tile, ts = 0, kb, ke;
  if (lo < hi) {
    ts = lo / KT;
    kb = lo - ts * KT;
    ke = min(KT, kb + hi - lo);
    lo += ke - kb;
    tile = n_whole + ts;
  } else {
    if (whole >= n_whole) break;
    tile = whole;
    whole += gridDim.x;
    kb = 0;
    ke = KT;
  }
  const int rb = tile % RB, cb = tile / RB;
  const int mt0 = rb * AF;
  if (!first) __syncthreads();  // every wave has read its last operands of the ring
  first = false;

  // this thread's share of a K step: unit u = q*64*NW + tid is fragment
  // q*NW + wave (wave-uniform), lane u%64
  const u32x4* src[LPT];
  size_t kstride[LPT];
#pragma unroll
  for (int q = 0; q < LPT; ++q) {
    const int f = q * NW + wave;
    if (f < NA) {
      const int mt = min(mt0 + (f % AF), a.MTtot - 1);  // rows past the operand: any valid tile
      src[q] = (const u32x4*)(f < AF ? a.Ahi : a.Alo) + (size_t)mt * 64 + lane;
      kstride[q] = (size_t)a.MTtot * 64;
    } else {
      const int st = cb * WF + (f - NA);
      src[q] = (const u32x4*)a.W + (size_t)(st >> 2) * a.wg + (size_t)(st & 3) * 64 + lane;
      kstride[q] = a.wk;
    }
  }
  // copy K step kt into ring slot `slot`: lane l's 16 bytes land at
  // sbuf[slot][f][l].  Steps past the range re-copy the last one, so every
  // iteration issues the same number of copies (constant vmcnt targets).
  auto issue = [&](int slot, int kt) __attribute__((always_inline)) {
    kt = min(kt, ke - 1);
#pragma unroll
    for (int q = 0; q < LPT; ++q)
      __builtin_amdgcn_global_load_lds((const void*)(src[q] + (size_t)kt * kstride[q]),
                                       (lds_void*)&sbuf[slot][q * NW + wave][0], 16, 0, 0);
  };

  f32x16 acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // the operands of one 16-wide K sub-step, held in registers: read from LDS
  // one sub-step ahead so the reads overlap the MFMAs of the one before
  struct Ops {
    u32x4 ah[WM], al[HI_LO ? WM : 1], bw[WN];
  };
  auto read_ops = [&](int buf, int s, Ops& o) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      o.ah[i] = sbuf[buf][wy * 2 * WM + 2 * i + fo][fl + 32 * s];
      if constexpr (HI_LO) o.al[i] = sbuf[buf][AF + wy * 2 * WM + 2 * i + fo][fl + 32 * s];
    }
#pragma unroll
    for (int j = 0; j < WN; ++j) o.bw[j] = sbuf[buf][NA + wx * 2 * WN + 2 * j + fo][fl + 32 * s];
  };
  // the MFMAs of one sub-step; the first one goes out before `between` (the
  // next sub-step's LDS reads), so the register wait it needs covers only the
  // previous reads, and the new reads overlap the remaining MFMAs
  auto mfma_ops = [&](const Ops& o, auto&& between) __attribute__((always_inline)) {
    acc[0][0] = mfma32_f16(o.ah[0], o.bw[0], acc[0][0]);
    __builtin_amdgcn_sched_barrier(0);
    between();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        if (i != 0 || j != 0) acc[i][j] = mfma32_f16(o.ah[i], o.bw[j], acc[i][j]);
        if constexpr (HI_LO) acc[i][j] = mfma32_f16(o.al[i], o.bw[j], acc[i][j]);
      }
    __builtin_amdgcn_sched_barrier(0);
  };

  // Ring schedule: step j lives in slot j % ST.  Iteration i multiplies the
  // first half of step i (read in the previous iteration) while its second
  // half is read; then it waits until step i+1 has landed (own copies: vmcnt;
  // everyone's: barrier), refills the slot of step i-1 with step i+ST-1, and
  // multiplies the second half while the first half of step i+1 is read.
  const int nk = ke - kb;
  {
    Ops o0, o1;
#pragma unroll
    for (int st = 0; st < ST - 1; ++st) issue(st, kb + st);
    vm_wait<LPT * (ST - 2)>();
    block_barrier();
    read_ops(0, 0, o0);
    int slot = 0;  // step i's
    for (int i = 0; i < nk; ++i) {
      // The loop starts 4 bytes past a multiple of 8: where the instructions before
      // it put it on a multiple of 8, a 2048-row prefill chunk of the 8B shape
      // took 7% longer (4 layers: 5.46 against 5.88 ms, gate/up 779 against 833 us).
      __builtin_amdgcn_sched_barrier(0);
      asm volatile(".p2align 3\n\ts_nop 0");
      __builtin_amdgcn_sched_barrier(0);
      const int next = slot + 1 == ST ? 0 : slot + 1, prev = slot == 0 ? ST - 1 : slot - 1;
      mfma_ops(o0, [&]() { read_ops(slot, 1, o1); });
      vm_wait<LPT * (ST - 3)>();
      block_barrier();
      issue(prev, kb + i + ST - 1);
      mfma_ops(o1, [&]() { read_ops(next, 0, o0); });
      slot = next;
    }
  }
  vm_wait<0>();  // no copy may land after the ring is reused or released

  const int row_w = rb * BM + wy * 32 * WM;
  const int col_w = cb * BN + wx * 32 * WN;
  if (nk < KT) {
    // A tile shared by several workgroups: this one's part goes out in
    // lane-native order (float4 group g of accumulator (i, j) of lane l at
    // ((i*WN + j)*4 + g)*64 + l of the wave's slice); tiled_finish sums a
    // tile's parts and runs the epilogue.
    float4* mine = (float4*)(a.part + ((size_t)(slot0 + ts) * NW + wave) * (size_t)(16 * WM * WN * 64));
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          mine[((i * WN + j) * 4 + g) * 64 + lane] =
              float4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
    continue;
  }
  __syncthreads();  // every wave has read its last operands: the ring becomes the epilogue's
  float* lds = (float*)&sbuf[0][0][0] + wave * (kEpiBytes / 4);
  EpiX<EPI> ex[2];
  epi_load_x<EPI>(a, row_w, col_w, ex[0]);
  // the block index is a compile-time constant, so the accumulators are
  // never indexed at run time (a rolled loop would move them to scratch)
  static_for<0, WM * WN / 2>([&](auto bc) {
    constexpr int blk = decltype(bc)::value, i = blk / (WN / 2), j = blk % (WN / 2) * 2;
    if constexpr (blk + 1 < WM * WN / 2) {
      constexpr int i1 = (blk + 1) / (WN / 2), j1 = (blk + 1) % (WN / 2) * 2;
      epi_load_x<EPI>(a, row_w + 32 * i1, col_w + 32 * j1, ex[(blk + 1) & 1]);
    }
    epi_block<EPI>(a, acc[i][j], acc[i][j + 1], row_w + 32 * i, col_w + 32 * j, inv_rms, ex[blk & 1], lds);
  });
  }
}

// Sums the parts of the shared tiles in K order (the same order whatever ran
// when) and runs the epilogue: one wave per 32 x 64 block.  A kernel of its
// own so that the whole chip takes part: summed by the last workgroup of
// each tile to arrive, the parts of 64 tiles kept 192 CUs waiting (512 rows x
// 4096 columns, K 4096, four-way: 73 us against 46).
template <int WY, int WX, int WM, int WN, int EPI>
__global__ __launch_bounds__(256) void tiled_finish(GemmArgs a, const float* __restrict__ inv_rms, int RB, int CB,
                                                    int n_shared, int n_sk) {
  constexpr int NW = WY * WX, BPW = WM * WN / 2;  // blocks per wave tile
  constexpr int BM = 32 * WM * WY, BN = 32 * WN * WX;
  __shared__ float4 region[4][kEpiBytes / 16];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.x * 4 + wv;
  if (b >= n_shared * NW * BPW) return;
  const int blk = b % BPW, wave = b / BPW % NW, ts = b / (BPW * NW);
  const int tile = RB * CB - n_shared + ts, rb = tile % RB, cb = tile / RB;
  const int i = blk / (WN / 2), j = blk % (WN / 2) * 2;
  const int row0 = rb * BM + wave / WX * 32 * WM + 32 * i, col0 = cb * BN + wave % WX * 32 * WN + 32 * j;
  if (row0 >= a.M) return;
  const int KT = a.KT;
  const SharedRuns runs(n_shared, KT, n_sk);
  const int w0 = runs.holder(ts * KT), w1 = runs.holder(ts * KT + KT - 1);
  EpiX<EPI> ex;
  epi_load_x<EPI>(a, row0, col0, ex);
  f32x16 c[2];
#pragma unroll
  for (int e = 0; e < 16; ++e) c[0][e] = c[1][e] = 0.f;
  auto slice = [&](int w) {
    return (const float4*)(a.part + ((size_t)(runs.slot0(w) + ts) * NW + wave) * (size_t)(16 * WM * WN * 64)) + (i * WN + j) * 4 * 64 + lane;
  };
  // two parts' loads in flight at a time
  for (int w = w0; w <= w1; w += 2) {
    float4 x[2][8];
    const float4 *p0 = slice(w), *p1 = slice(min(w + 1, w1));
#pragma unroll
    for (int g = 0; g < 8; ++g) x[0][g] = p0[g * 64];
#pragma unroll
    for (int g = 0; g < 8; ++g) x[1][g] = p1[g * 64];
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (h == 0 || w + 1 <= w1) {
#pragma unroll
        for (int g = 0; g < 8; ++g) {
          c[g >> 2][4 * (g & 3)] += x[h][g].x;
          c[g >> 2][4 * (g & 3) + 1] += x[h][g].y;
          c[g >> 2][4 * (g & 3) + 2] += x[h][g].z;
          c[g >> 2][4 * (g & 3) + 3] += x[h][g].w;
        }
      }
  }
  epi_block<EPI>(a, c[0], c[1], row0, col0, inv_rms, ex, (float*)region[wv]);
}

// Inverse RMS of each row from its per-16-column sums of squares (one wave
// per row, fixed summation order).
__global__ __launch_bounds__(256) void row_inv_rms(const float* __restrict__ ss, int ss_n, int M, float inv_dim,
                                                   float eps, float* __restrict__ out) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= M) return;
  float s = 0.f;
  for (int q = lane; q < ss_n; q += 64) s += ss[(size_t)row * ss_n + q];
  s = wave_sum(s);
  if (lane == 0) out[row] = rsqrtf(s * inv_dim + eps);
}

template <int WY, int WX, int WM, int WN, int EPI, bool HI_LO>
static hipError_t launch_t(const GemmArgs& a, const float* inv_rms, const TiledPlan& p, hipStream_t s) {
  const int BM = 32 * WM * WY, BN = 32 * WN * WX, NT = 64 * WY * WX;
  const int CB = a.NT * 16 / BN, RB = (a.MTtot * 16 + BM - 1) / BM;
  if (!tiled_plan_ok(p, CB * RB, a.KT))
    return hipErrorInvalidValue;
  hvd_launch((gemm_tiled<WY, WX, WM, WN, EPI, HI_LO>), dim3(p.n_wg), dim3(NT), 0, s, a, inv_rms, RB, CB, p.n_shared,
             p.n_sk);
  if (p.n_shared)
    hvd_launch((tiled_finish<WY, WX, WM, WN, EPI>), dim3((p.n_shared * WY * WX * WM * WN / 2 + 3) / 4), dim3(256), 0, s,
               a, inv_rms, RB, CB, p.n_shared, p.n_sk);
  return hipGetLastError();
}

template <int EPI, bool HI_LO>
static hipError_t launch_th(const GemmArgs& a, const float* inv_rms, const TiledPlan& p, hipStream_t s) {
  switch (p.tile) {
    case 0: return launch_t<2, 2, 2, 2, EPI, HI_LO>(a, inv_rms, p, s);  // 128 x 128, 4 waves
    case 1: return launch_t<2, 2, 2, 4, EPI, HI_LO>(a, inv_rms, p, s);  // 128 x 256, 4 waves
    case 2: return launch_t<4, 2, 2, 4, EPI, HI_LO>(a, inv_rms, p, s);  // 256 x 256, 8 waves
    case 3: return launch_t<2, 2, 4, 4, EPI, HI_LO>(a, inv_rms, p, s);  // 256 x 256, 4 waves
    case 4: return launch_t<2, 4, 2, 2, EPI, HI_LO>(a, inv_rms, p, s);  // 128 x 256, 8 waves
  }
  return hipErrorInvalidValue;
}

template <int EPI>
static hipError_t launch_te(const GemmArgs& a, const float* inv_rms, const TiledPlan& p, bool hi_lo, hipStream_t s) {
  return hi_lo ? launch_th<EPI, true>(a, inv_rms, p, s) : launch_th<EPI, false>(a, inv_rms, p, s);
}

hipError_t launch_gemm_tiled(int epi, const GemmArgs& a, const TiledPlan& p, bool hi_lo, float* inv_rms,
                             hipStream_t s) {
  if (epi != EPI_RESID) {
    const int rows = a.MTtot * 16;
    hvd_launch(row_inv_rms, dim3((rows + 3) / 4), dim3(256), 0, s, a.ss, a.ss_n, rows, a.inv_dim, a.eps,
                       inv_rms);
  }
  switch (epi) {
    case EPI_QKV: return launch_te<EPI_QKV>(a, inv_rms, p, hi_lo, s);
    case EPI_RESID: return launch_te<EPI_RESID>(a, inv_rms, p, hi_lo, s);
    case EPI_SILU: return launch_te<EPI_SILU>(a, inv_rms, p, hi_lo, s);
    case EPI_LM: return launch_te<EPI_LM>(a, inv_rms, p, hi_lo, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace hvd
