// GEMMs of 33 to 128 verify rows (gfx950, MFMA 16x16x32 f16): token trees,
// long drafts and small batches, where the weights still stream from HBM once
// but every weight fragment meets 3 to 8 row tiles.
//
// Bound: the weights' HBM stream, if the activations keep out of its way.
// Where every wave of gemm_skinny walks its own K steps, no two waves share an
// activation fragment: at five row tiles on the hi + lo pair each 4 KB of
// weights brings 10 KB of activations into registers, and each row tile costs
// about 4 us per launch.  Here the waves of a workgroup own columns instead:
//  * four waves each stream the weights of NSW strips of 16 columns into
//    registers, QD K steps ahead, and keep their accumulators for all the
//    rows: no reduction across waves;
//  * four more waves copy the activations, once per workgroup, into a ring of
//    LDS slots (global_load_lds) that the first four read.  Loads return in
//    order within a wave: in the streaming waves the copies (L2 hits) would
//    wait behind the weights, and the ring would have to be as deep as the
//    weight queue (measured: five row tiles, gate/up 62 us with 64 KB of
//    weights in flight per CU).  One copying wave is not enough: a wave issues
//    a 1 KB load every 37 ns at best (measured on L2 hits: 27 bytes per ns
//    with one wave per CU, 97 with four, 107 with eight).
// One slot holds KS K steps (2 on the pair, 4 single-pass).  One barrier per
// slot: slot i has landed, and slot i - 1 has been read.
//
// What bounds it now: weights and activations together pass a CU's vector
// memory path at 30 to 39 bytes per ns, whatever their shares (copies that hit
// the L2 queue behind weights on their way from HBM), so wider blocks pay.
//
// Column blocks that do not fill the CUs split K.  Each split publishes its
// partial tile with write-through stores and counts its arrival; the last one
// sums the splits in order and runs the epilogue.  (A second kernel for the sum
// took 5 us against 4 to 8 here, but its launch cost more: 72-row steps of the
// 8B shape 5.70 against 5.58 ms.)
//
// Measured (8B shape, us per launch, gemm_skinny -> here): gate/up 42.7 -> 39.9
// at 33 rows, 49.2 -> 43.8 at 72; LM head 203 -> 185 and 256 -> 210; 72-row
// steps 5.80 -> 5.41 ms, 33-row trees 4.65 -> 4.37.
#include "common.h"
#include "kernels.h"

#include <type_traits>

namespace hvd {

constexpr int kMidWaves = 4, kMidThreads = 64 * 2 * kMidWaves;  // streaming waves; as many copy

// K steps of weights in flight per streaming wave (4 NSW registers each)
constexpr int mid_depth(int MT, int NSW) { return NSW == 1 ? 24 : MT >= 7 ? 12 : 16; }
constexpr int kMidSlots = 4;  // ring slots: the copies of two may be in flight

// Inputs of a thread's octets (residual stream and gains, or rotary factors),
// requested before the partial tiles are published or read.
template <int MT, int COLS, int EPI, int NT>
struct MidX {
  static constexpr bool ON = EPI == EPI_RESID || EPI == EPI_QKV;
  static constexpr int OCT = COLS / 8, RPP = NT / OCT, N = (MT * 16 + RPP - 1) / RPP;  // rows per pass, passes
  float4 x[ON ? N : 1][2], gain[2];
};
template <int MT, int COLS, int EPI, int NT>
__device__ __forceinline__ void mid_load_x(const GemmArgs& a, const RowMeta* rows, int cb, int row0,
                                           MidX<MT, COLS, EPI, NT>& e) {
  if constexpr (EPI == EPI_QKV) {
    using X = MidX<MT, COLS, EPI, NT>;
    const int C = cb * COLS + threadIdx.x % X::OCT * 8;
    // (v columns: any valid factors)
    const int j = C < a.q_cols + a.kv_cols ? (C < a.q_cols ? C : C - a.q_cols) % a.dh >> 1 : 0;
#pragma unroll
    for (int i = 0; i < X::N; ++i) {
      const int r = min((int)threadIdx.x / X::OCT + i * X::RPP, MT * 16 - 1);
      const float4* rp = (const float4*)(a.rope + (size_t)rows[r].pos * (a.dh >> 1) + j);
      e.x[i][0] = rp[0];
      e.x[i][1] = rp[1];
    }
  }
  if constexpr (EPI == EPI_RESID) {
    using X = MidX<MT, COLS, EPI, NT>;
    const int C = cb * COLS + threadIdx.x % X::OCT * 8;
    e.gain[0] = *(const float4*)(a.gain_next + C);
    e.gain[1] = *(const float4*)(a.gain_next + C + 4);
#pragma unroll
    for (int i = 0; i < X::N; ++i) {
      const float4* xp = (const float4*)(a.X + (size_t)min(row0 + (int)threadIdx.x / X::OCT + i * X::RPP, a.M - 1) * a.D + C);
      e.x[i][0] = xp[0];
      e.x[i][1] = xp[1];
    }
  }
}

// Fused epilogue on the reduced tile (LDS, row pitch P floats): octets of 8
// columns of one row, 16 bytes per store where the output allows it.
template <int MT, int COLS, int EPI, int NT>
__device__ __forceinline__ void mid_epilogue(const GemmArgs& a, const float* tile, const float* inv_rms,
                                             const RowMeta* rows, int cb, int row0, const MidX<MT, COLS, EPI, NT>& ex) {
  constexpr int P = COLS + 4;
  const int tid = threadIdx.x;
  auto oct = [&](int r, int c, float (&v)[8]) __attribute__((always_inline)) {
    const float4 x = *(const float4*)(tile + r * P + c), y = *(const float4*)(tile + r * P + c + 4);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
  };
  if constexpr (EPI == EPI_RESID) {
    using E = MidX<MT, COLS, EPI, NT>;
    constexpr int OCT = E::OCT, RPP = E::RPP, N = E::N;
    const int o = tid % OCT, C = cb * COLS + o * 8;
    const float gn[8] = {ex.gain[0].x, ex.gain[0].y, ex.gain[0].z, ex.gain[0].w,
                         ex.gain[1].x, ex.gain[1].y, ex.gain[1].z, ex.gain[1].w};
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int r = tid / OCT + i * RPP, R = row0 + r;
      float v[8], n[8], sq = 0.f;
      oct(min(r, MT * 16 - 1), o * 8, v);
      v[0] += ex.x[i][0].x; v[1] += ex.x[i][0].y; v[2] += ex.x[i][0].z; v[3] += ex.x[i][0].w;
      v[4] += ex.x[i][1].x; v[5] += ex.x[i][1].y; v[6] += ex.x[i][1].z; v[7] += ex.x[i][1].w;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sq += v[e] * v[e];
        n[e] = v[e] * gn[e];
      }
      sq += __shfl_xor(sq, 1);  // the strip's other octet
      if (r < MT * 16 && R < a.M) {
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
    // strips in (gate, up) pairs: 16 act columns per pair
    constexpr int OCT = COLS / 16;
    for (int e = tid; e < MT * 16 * OCT; e += NT) {
      const int r = e / OCT, o = e % OCT, R = row0 + r;
      const int c = 32 * (o >> 1) + 8 * (o & 1);
      const float ir = inv_rms[r];
      float g[8], u[8];
      oct(r, c, g);
      oct(r, c + 16, u);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float v = g[i] * ir;
        u[i] = v / (1.f + __expf(-v)) * (u[i] * ir);
      }
      if (R < a.M) {
        uint4 hi, lo;
        split8(u, hi, lo);
        const size_t off = afrag_off(R, cb * (COLS / 2) + o * 8, a.MTtot);
        *(uint4*)(a.act_hi + off) = hi;
        *(uint4*)(a.act_lo + off) = lo;
      }
    }
  } else if constexpr (EPI == EPI_QKV) {
    using E = MidX<MT, COLS, EPI, NT>;
    const int o = tid % E::OCT, C = cb * COLS + o * 8;
#pragma unroll
    for (int i = 0; i < E::N; ++i) {
      const int r = tid / E::OCT + i * E::RPP, R = row0 + r;
      if (r >= MT * 16 || R >= a.M) continue;
      const RowMeta rm = rows[r];
      const float ir = inv_rms[r];
      _Float16* const page = a.kv + (size_t)(rm.kvs / kPage) * a.page_stride;
      const int slot = rm.kvs & (kPage - 1);
      float v[8];
      oct(r, o * 8, v);
      if (C < a.q_cols + a.kv_cols) {  // q and k: rotary pairs are adjacent columns
        const int base = C < a.q_cols ? 0 : a.q_cols;
        const int hg = (C - base) / a.dh, dp = (C - base) % a.dh;
        const float4 ca = ex.x[i][0], cb4 = ex.x[i][1];
        const float cc[4] = {ca.x, ca.z, cb4.x, cb4.z}, sn[4] = {ca.y, ca.w, cb4.y, cb4.w};
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float v0 = v[2 * e] * ir, v1 = v[2 * e + 1] * ir;
          w[e] = pack_h2(v0 * cc[e] - v1 * sn[e], v1 * cc[e] + v0 * sn[e]);
        }
        _Float16* dst = C < a.q_cols ? a.Q + (size_t)R * a.q_cols + C
                                     : page + ((size_t)hg * kPage + slot) * a.dh + dp;
        *(uint4*)dst = uint4{w[0], w[1], w[2], w[3]};
      } else {  // V is [dim][16 positions] in a page
        const int cv = C - a.q_cols - a.kv_cols;
        _Float16* vp = page + (size_t)a.Hkv * kPage * a.dh + (size_t)cv * kPage + slot;  // (head * dh + dim) * 16
#pragma unroll
        for (int e = 0; e < 8; ++e) vp[e * kPage] = (_Float16)(v[e] * ir);
      }
    }
  } else {  // EPI_LM: logits, and per row the max / lowest argmax over the block's columns
    constexpr int OCT = COLS / 8;
    static_assert(MT * 16 * OCT % 64 == 0, "whole waves in the last pass");
    for (int e = tid; e < MT * 16 * OCT; e += NT) {
      const int r = e / OCT, o = e % OCT, R = row0 + r, C = cb * COLS + o * 8;
      const float ir = inv_rms[r];
      float v[8], best = -INFINITY;
      int bidx = 0x7fffffff;
      oct(r, o * 8, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        v[i] *= ir;
        if (v[i] > best) {  // columns ascend: ties keep the lower one
          best = v[i];
          bidx = C + i;
        }
      }
#pragma unroll
      for (int s = 1; s < OCT; s <<= 1) {
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
          a.part_val[(size_t)R * a.n_part + cb] = best;
          a.part_idx[(size_t)R * a.n_part + cb] = bidx;
        }
      }
    }
  }
}

// Per-row sums of squares -> inverse RMS, by the copying waves (thread t of
// 256): 16 lanes per row, four 16-byte loads each in flight (rows of up to 4096
// columns; wider ones read the rest after).
template <int MT>
struct MidSS {
  float4 v[MT][4];
};
template <int MT>
__device__ __forceinline__ void mid_ss_issue(const GemmArgs& a, int t, int row0, MidSS<MT>& s) {
  const int r = t >> 4, j = t & 15, nq = a.ss_n >> 2;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const float4* p = (const float4*)(a.ss + (size_t)min(row0 + m * 16 + r, a.MTtot * 16 - 1) * a.ss_n);
#pragma unroll
    for (int i = 0; i < 4; ++i) s.v[m][i] = p[min(j + 16 * i, nq - 1)];
  }
}
template <int MT>
__device__ __forceinline__ void mid_ss_commit(const GemmArgs& a, int t, int row0, const MidSS<MT>& s, float* inv_rms) {
  const int r = t >> 4, j = t & 15, nq = a.ss_n >> 2;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 x = s.v[m][i];
      if (j + 16 * i < nq) sum += (x.x + x.y) + (x.z + x.w);
    }
    const float4* p = (const float4*)(a.ss + (size_t)min(row0 + m * 16 + r, a.MTtot * 16 - 1) * a.ss_n);
    for (int q = j + 64; q < nq; q += 16) {
      const float4 x = p[q];
      sum += (x.x + x.y) + (x.z + x.w);
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) sum += __shfl_xor(sum, o);
    if (j == 0) inv_rms[m * 16 + r] = rsqrtf(sum * a.inv_dim + a.eps);
  }
}

// Grid: n_cb column blocks x nsplit K splits x row blocks of MT tiles.
template <int MT, int NSW, int EPI, bool HL>
__global__ __launch_bounds__(kMidThreads, 2) void gemm_mid(GemmArgs a, int n_cb, int nsplit) {
  constexpr int KS = HL ? 2 : 4, HLN = HL ? 2 : 1;  // K steps per slot, parts of the activation
  constexpr int QD = mid_depth(MT, NSW), ST = kMidSlots;
  constexpr int FR = 4 * MT;                        // fragments per slot
  constexpr int COLS = 16 * NSW * kMidWaves, ROWS = 16 * MT, P = COLS + 4;
  static_assert(FR == KS * HLN * MT && QD % KS == 0, "whole slots");
  constexpr bool NORM = EPI != EPI_RESID;
  __shared__ u32x4 ring[ST * FR * 64];
  __shared__ float inv_rms[NORM ? ROWS : 1];
  __shared__ RowMeta rows[EPI == EPI_QKV ? ROWS : 1];
  static_assert(ROWS * P * 4 <= (int)sizeof(ring), "the tile fits the ring");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int split = blockIdx.x % nsplit, unit = blockIdx.x / nsplit;
  const int cb = unit % n_cb, mt0 = unit / n_cb * MT;
  // this split's K steps, in whole slots (the operand's last may be short)
  const int slots = (a.KT + KS - 1) / KS;
  const int s0 = (int)((int64_t)slots * split / nsplit), s1 = (int)((int64_t)slots * (split + 1) / nsplit);
  const int kb = s0 * KS, ke = min(a.KT, s1 * KS), n = s1 - s0;
  f32x4 acc[MT][NSW];

  // Every address below is a wave-uniform base, a 32-bit K offset (the host
  // checks that they fit) and the lane.
  if (wave >= kMidWaves) {
    MidSS<NORM ? MT : 1> ss;
    if constexpr (NORM) mid_ss_issue<MT>(a, tid - 64 * kMidWaves, mt0 * 16, ss);
    int4 rm{};
    if constexpr (EPI == EPI_QKV)
      rm = *(const int4*)(a.rows + min(mt0 * 16 + min(tid - 64 * kMidWaves, ROWS - 1), a.M - 1));
    const uint32_t astride = (uint32_t)a.MTtot * 1024;
    // this wave's fragments q * 4 + wave of a slot: K step, part (hi, lo), row tile
    const char* abase[MT];
    int aks[MT];
#pragma unroll
    for (int q = 0; q < MT; ++q) {
      const int f = q * kMidWaves + wave - kMidWaves, mt = f % MT, hl = f / MT % HLN;
      aks[q] = f / (MT * HLN);
      abase[q] = (const char*)(hl ? a.Alo : a.Ahi) + (size_t)min(mt0 + mt, a.MTtot - 1) * 1024;
    }
    auto copy = [&](int i) __attribute__((always_inline)) {
      u32x4* dst = &ring[(i % ST * FR + wave - kMidWaves) * 64];
#pragma unroll
      for (int q = 0; q < MT; ++q) {
        const char* p = abase[q] + (uint32_t)min(kb + i * KS + aks[q], ke - 1) * astride;
        __builtin_amdgcn_global_load_lds((const void*)(p + (uint32_t)lane * 16), (lds_void*)(dst + q * kMidWaves * 64), 16, 0, 0);
      }
    };
    // slots past the range re-read its last K step: one wait covers all
#pragma unroll
    for (int i = 0; i < ST - 1; ++i) copy(i);
    if constexpr (NORM) mid_ss_commit<MT>(a, tid - 64 * kMidWaves, mt0 * 16, ss, inv_rms);
    if constexpr (EPI == EPI_QKV)
      if (tid - 64 * kMidWaves < ROWS) rows[tid - 64 * kMidWaves] = RowMeta{rm.x, rm.y, rm.z, rm.w};
    for (int i = 0; i < n; ++i) {
      vm_wait<(ST - 2) * MT>();
      block_barrier();
      copy(i + ST - 1);
    }
    vm_wait<0>();  // no copy may land after the ring is reused
  } else {
    const uint32_t wstride = (uint32_t)a.wk * 16;
    const char* wbase[NSW];
#pragma unroll
    for (int j = 0; j < NSW; ++j) {
      const int st = (cb * kMidWaves + wave) * NSW + j;
      wbase[j] = (const char*)(a.W + (size_t)(st >> 2) * a.wg + (size_t)(st & 3) * 64);
    }
    u32x4 qw[QD][NSW];
    auto load_w = [&](int q, int k) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < NSW; ++j)
        qw[q][j] = __builtin_nontemporal_load((const u32x4*)(wbase[j] + (uint32_t)min(k, ke - 1) * wstride + (uint32_t)lane * 16));
    };
    // (K steps past the range re-read its last one, so that the first QD go
    // out without a branch: one would keep the compiler from counting them)
#pragma unroll
    for (int q = 0; q < QD; ++q) load_w(q, kb + q);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int j = 0; j < NSW; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const u32x4* base = ring + lane;
    int slot = 0;
    auto step = [&](int q, int ks) __attribute__((always_inline)) {
#pragma unroll
      for (int hl = 0; hl < HLN; ++hl)
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const u32x4 af = base[(slot * FR + (ks * HLN + hl) * MT + m) * 64];
#pragma unroll
          for (int j = 0; j < NSW; ++j) acc[m][j] = mfma_f16(af, qw[q][j], acc[m][j]);
        }
    };
    auto next_slot = [&]() __attribute__((always_inline)) {
      __builtin_amdgcn_sched_barrier(0);  // this slot's reads stay before the next barrier
      slot = slot + 1 == ST ? 0 : slot + 1;
    };
    int k = kb;
    for (; k + QD < ke; k += QD) {
#pragma unroll
      for (int q = 0; q < QD; ++q) {
        if (q % KS == 0) block_barrier();
        step(q, q % KS);
        load_w(q, k + q + QD);
        if (q % KS == KS - 1) next_slot();
      }
    }
    // at most QD steps are left, all in flight
#pragma unroll
    for (int q = 0; q < QD; q += KS) {
      if (k + q >= ke) break;
      block_barrier();
      if (k + q + KS <= ke) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) step(q + ks, ks);
      } else {  // the operand's last slot, cut short
#pragma unroll
        for (int ks = 0; ks + 1 < KS; ++ks)
          if (k + q + ks < ke) step(q + ks, ks);
      }
      next_slot();
    }
  }
  __syncthreads();  // every wave has read its last activations: the ring becomes the tile

  MidX<MT, COLS, EPI, kMidThreads> ex;
  mid_load_x<MT, COLS, EPI, kMidThreads>(a, rows, cb, mt0 * 16, ex);
  float* tile = (float*)ring;
  if (wave < kMidWaves) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int j = 0; j < NSW; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          tile[(m * 16 + 4 * (lane >> 4) + e) * P + (wave * NSW + j) * 16 + (lane & 15)] = acc[m][j][e];
  }
  __syncthreads();
  if (nsplit > 1) {
    constexpr int QPR = COLS / 4, TOTAL = ROWS * QPR, N = (TOTAL + kMidThreads - 1) / kMidThreads;  // float4 per thread
    float* part = a.part + (size_t)unit * nsplit * ROWS * COLS;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int e = q * kMidThreads + tid;
      if (e < TOTAL)
        st_f4_dev(part, (uint32_t)((split * ROWS * COLS + e * 4) * 4), *(const float4*)(tile + e / QPR * P + e % QPR * 4));
    }
    vm_wait<0>();  // this thread's stores are done
    __syncthreads();   // (and every thread has read its part of the tile)
    int* flag = (int*)tile;
    if (tid == 0) *flag = atomicAdd(a.cnt + unit, 1u) == (uint32_t)nsplit - 1u;
    __syncthreads();
    const bool last = *flag != 0;
    __syncthreads();
    if (!last) return;
    if (tid == 0) store_dev_u32(a.cnt + unit, 0u);  // ready for the next launch
    // As many loads in flight as registers allow (a round trip to the memory
    // side takes about 2 us), and none of them under a branch, which would wait
    // for those before it: parts past the last split re-read it.
    auto sum = [&](auto sb) __attribute__((always_inline)) {
      constexpr int SB = decltype(sb)::value, QB = N < 40 / SB ? N : 40 / SB;  // parts and float4 per batch
#pragma unroll
      for (int q = 0; q < N; q += QB) {
        float4 v[QB];
#pragma unroll
        for (int h = 0; h < QB; ++h) v[h] = float4{0.f, 0.f, 0.f, 0.f};
        for (int p0 = 0; p0 < nsplit; p0 += SB) {
          float4 t[QB][SB];
#pragma unroll
          for (int h = 0; h < QB; ++h)
#pragma unroll
            for (int p = 0; p < SB; ++p) {
              const int e = min((q + h) * kMidThreads + tid, TOTAL - 1);
              t[h][p] = ld_f4_dev(part, (uint32_t)((min(p0 + p, nsplit - 1) * ROWS * COLS + e * 4) * 4));
            }
#pragma unroll
          for (int h = 0; h < QB; ++h)
#pragma unroll
            for (int p = 0; p < SB; ++p) {
              const bool in = p0 + p < nsplit;
              v[h].x += in ? t[h][p].x : 0.f;
              v[h].y += in ? t[h][p].y : 0.f;
              v[h].z += in ? t[h][p].z : 0.f;
              v[h].w += in ? t[h][p].w : 0.f;
            }
        }
#pragma unroll
        for (int h = 0; h < QB; ++h) {
          const int e = (q + h) * kMidThreads + tid;
          if (q + h < N && e < TOTAL) *(float4*)(tile + e / QPR * P + e % QPR * 4) = v[h];
        }
      }
    };
    if (nsplit == 2) sum(std::integral_constant<int, 2>{});
    else if (nsplit <= 4) sum(std::integral_constant<int, 4>{});
    else sum(std::integral_constant<int, 8>{});
    __syncthreads();
  }
  mid_epilogue<MT, COLS, EPI, kMidThreads>(a, tile, inv_rms, rows, cb, mt0 * 16, ex);
}

template <int MT, int NSW, int EPI>
static hipError_t launch_mid(const GemmArgs& a, int splits, int mblocks, bool hi_lo, hipStream_t s) {
  const int n_cb = a.NT / (NSW * kMidWaves);
  const dim3 grid(n_cb * mblocks * splits);
  if (hi_lo) {
    hvd_launch((gemm_mid<MT, NSW, EPI, true>), grid, dim3(kMidThreads), 0, s, a, n_cb, splits);
  } else {
    if constexpr (EPI == EPI_QKV) return hipErrorInvalidValue;
    else hvd_launch((gemm_mid<MT, NSW, EPI, false>), grid, dim3(kMidThreads), 0, s, a, n_cb, splits);
  }
  return hipGetLastError();
}

template <int NSW, int EPI>
static hipError_t launch_mid_mt(const GemmArgs& a, int mt, int splits, int mblocks, bool hi_lo, hipStream_t s) {
  switch (mt) {
    case 3: return launch_mid<3, NSW, EPI>(a, splits, mblocks, hi_lo, s);
    case 4: return launch_mid<4, NSW, EPI>(a, splits, mblocks, hi_lo, s);
    case 5: return launch_mid<5, NSW, EPI>(a, splits, mblocks, hi_lo, s);
    case 6: return launch_mid<6, NSW, EPI>(a, splits, mblocks, hi_lo, s);
    case 7: return launch_mid<7, NSW, EPI>(a, splits, mblocks, hi_lo, s);
    case 8: return launch_mid<8, NSW, EPI>(a, splits, mblocks, hi_lo, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_mid(int epi, const GemmArgs& a, const MidPlan& p, bool hi_lo, hipStream_t s) {
  const int strips = p.strips, splits = p.splits, mblocks = p.mblocks, mt_block = p.mt_block;
  // what the kernel assumes: whole column blocks, K slots for every split,
  // partial offsets of one block within 32 bits
  if ((strips != 4 && strips != 8) || a.NT % strips || splits < 1 || mblocks < 1 || mblocks * mt_block < a.MTtot ||
      (mblocks - 1) * mt_block >= a.MTtot || a.X_out || splits > std::max(1, a.KT / 4) ||
      (int64_t)splits * mt_block * 16 * strips * 64 > INT32_MAX || (int64_t)a.MTtot * a.KT * 1024 > INT32_MAX ||
      (int64_t)a.wk * a.KT * 16 > INT32_MAX)
    return hipErrorInvalidValue;
  switch (epi) {
    case EPI_QKV: return strips == 8 ? launch_mid_mt<2, EPI_QKV>(a, mt_block, splits, mblocks, hi_lo, s) : launch_mid_mt<1, EPI_QKV>(a, mt_block, splits, mblocks, hi_lo, s);
    case EPI_RESID: return strips == 8 ? launch_mid_mt<2, EPI_RESID>(a, mt_block, splits, mblocks, hi_lo, s) : launch_mid_mt<1, EPI_RESID>(a, mt_block, splits, mblocks, hi_lo, s);
    case EPI_SILU: return strips == 8 ? launch_mid_mt<2, EPI_SILU>(a, mt_block, splits, mblocks, hi_lo, s) : launch_mid_mt<1, EPI_SILU>(a, mt_block, splits, mblocks, hi_lo, s);
    case EPI_LM: return strips == 8 ? launch_mid_mt<2, EPI_LM>(a, mt_block, splits, mblocks, hi_lo, s) : launch_mid_mt<1, EPI_LM>(a, mt_block, splits, mblocks, hi_lo, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace hvd
