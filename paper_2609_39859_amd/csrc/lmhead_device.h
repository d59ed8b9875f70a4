// Device code shared by the LM-head kernels: operand swizzle, tile mapping,
// accumulator layouts, the per-column statistics over the vocabulary and the
// drawing of candidates.  The bf16 kernels all take column_stats of the 128
// vocabulary rows a wave holds and merge2 of a tile's two halves, in this
// order, so the partials of a (position, tile) have the same bits whichever
// kernel computed them; the fp32 kernels likewise over eight waves' 32 rows.
#pragma once

#include "fork_kernels.h"

#include <math.h>

#include <type_traits>

namespace fork {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSlab = 128;                   // bytes of K per row per stage
constexpr int kOperandBytes = 256 * kSlab;   // 32 KiB: one operand, one stage
constexpr int kGroupV = 8;                   // vocab stripes per sweep group
constexpr int kXcds = 8;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
// Raw-buffer descriptor word 3 for gfx9-family buffers: 32-bit data format,
// offsets checked against the record count (out of range reads return 0).
constexpr int kBufferWord3 = 0x00020000;
constexpr unsigned kOutOfRange = 0x80000000u;

__device__ __forceinline__ int swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }

// Workgroup id `bid` of `n` in the order of its XCD: workgroups are dealt to the
// XCDs round-robin (XCD x gets x, x + 8, ...), each takes a contiguous range.
__device__ __forceinline__ int xcd_order(int bid, int n) {
  const int x = bid % kXcds, i = bid / kXcds;
  return x * (n / kXcds) + min(x, n % kXcds) + i;
}

// (vocabulary tile, position tile) of a place in the launch order.
__device__ __forceinline__ void tile_of(int logical, int nvt, int npt, int& vt, int& pt) {
  const int per_group = kGroupV * npt;
  const int group = logical / per_group;
  const int in = logical - group * per_group;
  const int gv0 = group * kGroupV;
  const int gvn = min(kGroupV, nvt - gv0);
  pt = in / gvn;
  vt = gv0 + (in - pt * gvn);
}

// Maps the hardware workgroup id (of the first n) to its tile.
__device__ __forceinline__ void map_tile(int bid, int n, int nvt, int npt, int& vt, int& pt) {
  tile_of(xcd_order(bid, n), nvt, npt, vt, pt);
}

// Merge of two partials (either may be empty, s == 0).
__device__ __forceinline__ float4 merge2(float4 a, float4 b) {
  if (b.y == 0.f) return a;
  if (a.y == 0.f) return b;
  const float m = fmaxf(a.x, b.x);
  const float ea = exp2f((a.x - m) * kLog2e), eb = exp2f((b.x - m) * kLog2e);
  float4 r;
  r.x = m;
  r.y = a.y * ea + b.y * eb;
  r.z = ea * (a.z + (a.x - m) * a.y) + eb * (b.z + (b.x - m) * b.y);
  const int ia = __float_as_int(a.w), ib = __float_as_int(b.w);
  const bool take_a = (a.x > b.x) || (a.x == b.x && ia < ib);
  r.w = __int_as_float(take_a ? ia : ib);
  return r;
}

// Philox4x32-10: ten rounds of the 4x32 S-box (two 32 x 32 -> 64-bit
// products whose halves are exchanged and mixed with the other counter words
// and the round key), the key advanced by the Weyl constants between rounds.
// Each product is one 32 x 32 -> 64-bit multiply (v_mad_u64_u32).
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
    c = make_uint4((uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1,
                   (uint32_t)(p0 >> 32) ^ c.w ^ k1, (uint32_t)p0);
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c;
}

// Gumbel key of one logit: z / tau - log E with E = -log(1 - U) and U on the
// odd grid (2 (w >> 9) + 1) 2^-24 of (0, 1).  1 - U is exact in binary32, so
// E comes from the hardware base-2 logarithm, except below U = 2^-7, where
// the series U + U^2/2 + U^3/3 + U^4/4 (relative error < U^4/5 < 2^-30)
// avoids the cancellation of a logarithm near 1.  The key carries a relative
// error of about 1e-6 in E, far below the logit rounding.
__device__ __forceinline__ float gumbel_key(float z, float inv_tau, uint32_t w) {
  const float u = (float)(2u * (w >> 9) + 1u) * 0x1p-24f;
  const float series = u * fmaf(u, fmaf(u, fmaf(u, 0.25f, 1.0f / 3.0f), 0.5f), 1.0f);
  const float viaLog = -__builtin_amdgcn_logf(1.0f - u) * kLn2;
  const float e = u < 0x1p-7f ? series : viaLog;
  return fmaf(z, inv_tau, -__builtin_amdgcn_logf(e) * kLn2);
}

// Accumulator layout: a lane's accumulators hold vocabulary values (MFMA rows)
// of whole positions (MFMA columns), so the reduction over the vocabulary is
// mostly in-lane.
//
// AccN (16 x 16 MFMA blocks): a wave's 16 I x 16 N outputs are I x N blocks of
// 16 x 16; element e of block (i, j) in lane l is row 16 i + 4 (l / 16) + e,
// column 16 j + l % 16.  The four lanes l % 16 + 16 g (g = 0..3) hold the rows
// of a column, 4 I each.
template <int N, int I = 8>
struct AccN {
  typedef f32x4 Arr[I][N];
  static constexpr int kNI = I, kNJ = N, kNE = 4;
  static constexpr int kRows = 16 * I;
  static constexpr int kLeaders = 16;  // lanes 0..15 hold one copy of each column
  __device__ static float get(const Arr& a, int i, int j, int e) { return a[i][j][e]; }
  __device__ static void set(Arr& a, int i, int j, int e, float v) { a[i][j][e] = v; }
  __device__ static int row(int i, int e, int lane) { return i * 16 + (lane >> 4) * 4 + e; }
  __device__ static int col(int j, int lane) { return j * 16 + (lane & 15); }
  // combine the copies of a column: lanes 16 and 32 apart
  template <class F>
  __device__ static void across(F&& f) {
    f(16);
    f(32);
  }
};
typedef AccN<4> Acc16;

// What the epilogue produces besides the per-tile statistics.
enum EpilogueMode { kGreedy = 0, kDrawn = 1, kTarget = 2 };

// Per-position inputs of the epilogue, loaded before the last MFMAs so that
// their latency is hidden: the given token (kTarget) or the draw's row index
// (kDrawn) of each column this lane holds.
template <class Lay>
struct ColIn {
  int col[Lay::kNJ];
};

// Launch position of column c (0..255) of position tile pt.  Contiguous:
// p0 + c.  Interleaved (M = 256 * npt, the drawing kernel over all rows):
// 16-column block k of tile pt is the 16-row chunk k * npt + (pt + k) mod
// npt, i.e. column c is row of that chunk's c % 16-th; chunk k * npt + s
// goes to tile (s - k) mod npt.  The active blocks, the only rows whose
// candidates are drawn, usually sit at a fixed offset in every sequence;
// the rotation by k spreads them over the position tiles instead of
// gathering them in a few (which a plain stride of npt chunks does whenever
// the sequence length is a multiple of 16 npt), so the tiles' epilogues
// cost about the same.
struct PosMap {
  int p0, pt, npt;
  bool ilv;
  __device__ int operator()(int c) const {
    const int k = c >> 4;
    return ilv ? ((k * npt + (pt + k) % npt) << 4) + (c & 15) : p0 + c;
  }
};

template <class Lay, int kMode>
__device__ __forceinline__ void load_col_inputs(ColIn<Lay>& ci, int tid, int lane, int wp,
                                                const PosMap& pos, int M, const SampleArgs& sa,
                                                const TargetArgs& ta) {
  if (kMode == kGreedy) return;
  const int32_t* src = kMode == kTarget ? ta.token : sa.row;
#pragma unroll
  for (int j = 0; j < Lay::kNJ; ++j) {
    const int p = pos(wp * 64 + Lay::col(j, lane));
    ci.col[j] = p < M ? src[p] : -1;
  }
}

// Statistics of the logits of column j that this lane holds (rows vbase +
// Lay::row(i, e, lane), increasing in (i, e)), combined with the lanes that
// hold the column's other rows: the maximum m, the lowest row holding it,
// s = sum e^(z-m) and t = sum e^(z-m)(z-m).  Branch-free.  Unless kFull
// (every row < V), rows past V are set to -inf in acc first, so that no pass
// needs a row test.
template <class Lay, bool kFull>
__device__ __forceinline__ void column_stats(typename Lay::Arr& acc, int j, int lane, int vbase,
                                             int V, float& m_out, int& idx_out, float& s_out,
                                             float& t_out) {
  if (!kFull) {
#pragma unroll
    for (int i = 0; i < Lay::kNI; ++i)
#pragma unroll
      for (int e = 0; e < Lay::kNE; ++e)
        if (vbase + Lay::row(i, e, lane) >= V) Lay::set(acc, i, j, e, -INFINITY);
  }
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < Lay::kNI; ++i)
#pragma unroll
    for (int e = 0; e < Lay::kNE; ++e) m = fmaxf(m, Lay::get(acc, i, j, e));
  // the lowest row holding m: scan from the highest row down
  int idx = 0x7fffffff;
#pragma unroll
  for (int i = Lay::kNI - 1; i >= 0; --i)
#pragma unroll
    for (int e = Lay::kNE - 1; e >= 0; --e)
      idx = Lay::get(acc, i, j, e) == m ? vbase + Lay::row(i, e, lane) : idx;
  Lay::across([&](int off) {
    const float mo = __shfl_xor(m, off);
    const int io = __shfl_xor(idx, off);
    const bool take = mo > m || (mo == m && io < idx);
    m = take ? mo : m;
    idx = take ? io : idx;
  });
  float s = 0.f, tl = 0.f;
  // with few rows per lane the sums are taken without a branch, so that the
  // columns' chains of exchanges can overlap
  constexpr bool kBranch = Lay::kNI > 2;
  if (!kBranch || m > -INFINITY) {
    const float nml = -m * kLog2e;
#pragma unroll
    for (int i = 0; i < Lay::kNI; ++i)
#pragma unroll
      for (int e = 0; e < Lay::kNE; ++e) {
        // (z - m) * log2(e) with one rounding; the moment is summed in
        // these units and scaled by ln 2 once
        const float dl = fmaf(Lay::get(acc, i, j, e), kLog2e, nml);
        const float ex = __builtin_amdgcn_exp2f(dl);
        s += ex;
        // a -inf row has ex = 0: keep 0 * -inf out of the moment
        tl = fmaf(ex, kFull ? dl : fmaxf(dl, -1e30f), tl);
      }
  }
  // lanes holding the same column add in the same order: identical results
  Lay::across([&](int off) {
    s += __shfl_xor(s, off);
    tl += __shfl_xor(tl, off);
  });
  m_out = m;
  idx_out = idx;
  s_out = kBranch || m > -INFINITY ? s : 0.f;
  t_out = kBranch || m > -INFINITY ? tl * kLn2 : 0.f;
}

// The logit of row tk (a given token) in column j, if this lane holds it among
// the wave's rows from vbase.
template <class Lay>
__device__ __forceinline__ bool column_target(const typename Lay::Arr& acc, int j, int lane,
                                              int vbase, int V, int tk, float& z) {
  if (tk < vbase || tk >= vbase + Lay::kRows || tk >= V) return false;
  bool hit = false;
#pragma unroll
  for (int i = 0; i < Lay::kNI; ++i)
#pragma unroll
    for (int e = 0; e < Lay::kNE; ++e)
      if (vbase + Lay::row(i, e, lane) == tk) {
        z = Lay::get(acc, i, j, e);
        hit = true;
      }
  return hit;
}

// Drawn-candidate partials {key, idx bits, z, 0}: larger key wins, lower
// index on equal keys.
__device__ __forceinline__ float4 pick_drawn(float4 a, float4 b) {
  const bool take_a = a.x > b.x || (a.x == b.x && __float_as_int(a.y) < __float_as_int(b.y));
  return make_float4(take_a ? a.x : b.x, take_a ? a.y : b.y, take_a ? a.z : b.z, 0.f);
}

// The maximiser of the Gumbel keys of column j over the wave's rows from vbase,
// for the lanes whose column is drawn (srow >= 0): best key, its lowest row
// and its logit, combined over the lanes holding the column.  Rows past V hold
// -inf (column_stats), whose key is never taken, so a ragged tile needs no row
// test; blocks wholly past V are skipped.  (With a test per row a launch whose
// time is that of its ragged tiles took longer: M = 2739, d = 272, V = 5491,
// drawn over all rows 28.2 -> 26.2 us, V = 5632, which has none, 24.1 -> 23.8.)
template <class Lay, bool kFull>
__device__ __forceinline__ void column_draw(const typename Lay::Arr& acc, int j, int lane,
                                            int vbase, int V, int srow, const SampleArgs& sa,
                                            float& best, int& bidx, float& bz) {
  best = -INFINITY;
  bz = 0.f;
  bidx = 0x7fffffff;
  if (srow >= 0) {
    // elements 4g .. 4g + 3 of a block are four consecutive rows from
    // a multiple of 4: one generator call yields their four words
#pragma unroll
    for (int i = 0; i < Lay::kNI; ++i) {
      if (!kFull && vbase + 16 * i >= V) break;
#pragma unroll
      for (int g = 0; g < Lay::kNE / 4; ++g) {
        const int vq = vbase + Lay::row(i, 4 * g, lane);
        const uint4 w = philox4x32_10(
            make_uint4((uint32_t)vq >> 2, (uint32_t)srow, sa.counter, 0u), sa.key0, sa.key1);
        const uint32_t words[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float z = Lay::get(acc, i, j, 4 * g + c);
          const float key = gumbel_key(z, sa.inv_tau, words[c]);
          if (key > best) {
            best = key;
            bidx = vq + c;
            bz = z;
          }
        }
      }
    }
  }
  Lay::across([&](int off) {
    const float ob = __shfl_xor(best, off), oz = __shfl_xor(bz, off);
    const int oi = __shfl_xor(bidx, off);
    if (ob > best || (ob == best && oi < bidx)) {
      best = ob;
      bidx = oi;
      bz = oz;
    }
  });
}

__device__ __forceinline__ void barrier_nofence() {
  // s_barrier alone: the release fence of __syncthreads would also wait for
  // the loads still in flight for later stages.  The empty asm statements
  // keep the compiler from moving LDS accesses across the barrier.
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// s_waitcnt with vmcnt <= n and lgkmcnt == 0 (expcnt not waited on).
template <int N>
__device__ __forceinline__ void wait_vm_lgkm0() {
  static_assert(N >= 0 && N < 64, "vmcnt field");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
}

}  // namespace
}  // namespace fork
