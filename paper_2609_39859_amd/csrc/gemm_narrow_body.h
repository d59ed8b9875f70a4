// The body of the LM head with 64 NJ positions per workgroup (bf16): see
// gemm_narrow.hip for its design and what it measured.
#pragma once

#include "lmhead_device.h"

namespace fork {
namespace {

constexpr int kWaves = 8;                   // 2 vocabulary halves x 4 position quarters
constexpr int kHSlots = 2;                  // hidden ring
constexpr int kNontemporal = 2;             // cache policy bits of a buffer load

constexpr int narrow_lds_bytes(int NJ, int WS) {
  return WS * kOperandBytes + kHSlots * 64 * NJ * kSlab;
}

// One workgroup of 512 threads: vocabulary tile vt, positions p0 .. p0 + 64 NJ,
// W ring of WS = 3 slots (W two stages ahead of its use) or 2 (one stage, with
// 80 KiB for NJ = 1, so that two workgroups share a CU), smem of
// narrow_lds_bytes(NJ, WS).
template <int NJ, bool kNt, int kMode, int WS>
__device__ __forceinline__ void gemm_narrow_body(
    unsigned char* smem, const unsigned char* __restrict__ hidden,
    const unsigned char* __restrict__ W, int M, int d, int V, int vt, int p0,
    float4* __restrict__ partials, const int32_t* __restrict__ rowlist, int Mh,
    const SampleArgs& sa, const TargetArgs& ta) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the name
  typedef AccN<NJ> Lay;
  constexpr int kWaveP = 16 * NJ;        // positions per wave
  constexpr int kTP = 4 * kWaveP;        // positions per workgroup
  constexpr int LW = 4, LH = NJ;         // loads of a wave per stage
  constexpr int kHBytes = kTP * kSlab;   // hidden, one stage
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wv = wave & 1;   // vocabulary half: rows wv*128 .. +128
  const int wp = wave >> 1;  // position quarter

  const int v0 = vt * kTileV;

  const int row_bytes = d * 2;
  const int kchunks = row_bytes >> 4;  // 16-byte chunks per row
  const int nk = (kchunks + 7) >> 3;   // 128-byte stages
  const int kfull = kchunks >> 3;      // stages whose chunks all lie inside d

  // Rows past the end of W / hidden lie outside the record counts and read as
  // zero; with a row list the hidden descriptor spans all Mh rows.
  const bool listed = rowlist != nullptr;
  const unsigned recW = (unsigned)(min(kTileV, V - v0) * row_bytes);
  const unsigned recH =
      listed ? (unsigned)(Mh * row_bytes) : (unsigned)(min(kTP, M - p0) * row_bytes);
  const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(W + (size_t)v0 * row_bytes), (short)0, (int)recW, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rsH = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(hidden + (listed ? (size_t)0 : (size_t)p0 * row_bytes)), (short)0, (int)recH,
      kBufferWord3);

  // A load instruction of a wave fills 1 KiB of LDS, 8 rows x 128 B: lane l
  // the chunk slot l % 8 of row l / 8, so it loads the logical chunk kept
  // there (8-row groups with an odd number have bit 0 of the chunk flipped).
  const int lrow = lane >> 3;
  auto chunk = [&](int group) { return (lane & 7) ^ lrow ^ (group & 1); };
  unsigned woff[LW], hoff[LH];
#pragma unroll
  for (int q = 0; q < LW; ++q) {
    const int g = wave * LW + q;
    woff[q] = (unsigned)((g * 8 + lrow) * row_bytes) + (unsigned)(chunk(g) << 4);
  }
#pragma unroll
  for (int q = 0; q < LH; ++q) {
    const int g = wave * LH + q, p = g * 8 + lrow;  // p: position within the tile
    int r = p;
    if (listed) {
      r = p0 + p < M ? rowlist[p0 + p] : -1;
      if (r >= Mh) r = -1;
    }
    hoff[q] = r >= 0 ? (unsigned)(r * row_bytes) + (unsigned)(chunk(g) << 4) : kOutOfRange;
  }
  // Offset of a load in stage s; chunks past d, and stages past the end, lie
  // beyond every record count.
  auto at = [&](unsigned off, int s, int group) -> unsigned {
    const bool in = s < kfull || s * 8 + chunk(group) < kchunks;
    return in && off != kOutOfRange ? off + (unsigned)(s * kSlab) : kOutOfRange;
  };
  auto issue_W1 = [&](int s, int slot, int q) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rsW,
        (__attribute__((address_space(3))) void*)(smem + slot * kOperandBytes +
                                                  (wave * LW + q) * 1024),
        16, at(woff[q], s, wave * LW + q), 0, 0, kNt ? kNontemporal : 0);
  };
  auto issue_H1 = [&](int s, int slot, int q) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rsH,
        (__attribute__((address_space(3))) void*)(smem + WS * kOperandBytes + slot * kHBytes +
                                                  (wave * LH + q) * 1024),
        16, at(hoff[q], s, wave * LH + q), 0, 0, 0);
  };

  typename Lay::Arr acc;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // Fragments of step kk of a stage: chunk 2 kq + kk of the rows, kq = lane / 16.
  const int fr = lane & 15;
  const int kq = lane >> 4;
  const int fx = swz(fr);
  auto rd_a = [&](int slot, int kk, int i) {
    return *reinterpret_cast<const bf16x8*>(smem + slot * kOperandBytes +
                                            (wv * 128 + fr + 16 * i) * kSlab +
                                            (((2 * kq + kk) ^ fx) << 4));
  };
  auto rd_b = [&](int slot, int kk, int j) {
    return *reinterpret_cast<const bf16x8*>(smem + WS * kOperandBytes + slot * kHBytes +
                                            (wp * kWaveP + fr + 16 * j) * kSlab +
                                            (((2 * kq + kk) ^ fx) << 4));
  };

  // The given token (kTarget) or draw row (kDrawn) of each column of this lane.
  int col_in[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int p = p0 + wp * kWaveP + Lay::col(j, lane);
    const int32_t* src = kMode == kTarget ? ta.token : sa.row;
    col_in[j] = kMode != kGreedy && p < M ? src[p] : -1;
  }

  // kLive: the wave's positions include one below M; other waves only load
  // their share of each stage and take each barrier.
  auto mainloop = [&](auto live_tag) {
    constexpr bool kLive = decltype(live_tag)::value;
    bf16x8 a[8], b0[NJ], b1[NJ];
    auto mfma_row = [&](int i, const bf16x8(&b)[NJ]) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    };
    // Load order W0 H0 W1 H1, then per stage k: W(k + 2) in the first step
    // (WS = 3), H(k + 2) (WS = 2: and W(k + 2)) in the second, after the stage's
    // barrier.  At that barrier only W(k + 2) (WS = 2: nothing) may be in
    // flight; every slot refilled after it belongs to a
    // stage whose fragments all waves have read.
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int q = 0; q < LW; ++q) issue_W1(s, s, q);
#pragma unroll
      for (int q = 0; q < LH; ++q) issue_H1(s, s, q);
    }
    wait_vm_lgkm0<LW + LH>();
    barrier_nofence();
    if (kLive) {
#pragma unroll
      for (int i = 0; i < 8; ++i) a[i] = rd_a(0, 0, i);
#pragma unroll
      for (int j = 0; j < NJ; ++j) b0[j] = rd_b(0, 0, j);
    }
    int ws = 0, hs = 0, ws2 = 2;  // W slots of stages k and k + 2, hidden slot of k
    for (int k = 0; k < nk; ++k) {
      const int ws1 = ws == WS - 1 ? 0 : ws + 1, hs1 = hs ^ 1;
      // first step; after the MFMAs of row i its fragment is refilled for the
      // second step
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (kLive) {
          mfma_row(i, b0);
          a[i] = rd_a(ws, 1, i);
          if (i < NJ) b1[i] = rd_b(hs, 1, i);
        }
        if (WS == 3 && (i & 1)) issue_W1(k + 2, ws2, i >> 1);
      }
      if (kLive) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, NJ, 0);  // MFMA
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read
          if (i < NJ) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          if (WS == 3 && (i & 1)) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // load
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      // second step; the barrier after its first two rows, so that queued
      // MFMAs cover it, and the next stage's fragments after the barrier
      if (kLive) {
        mfma_row(0, b1);
        mfma_row(1, b1);
      }
      __builtin_amdgcn_sched_barrier(0);
      wait_vm_lgkm0<WS == 3 ? LW : 0>();
      barrier_nofence();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 2; i < 8; ++i) {
        if (kLive) {
          mfma_row(i, b1);
          a[i] = rd_a(ws1, 0, i);
          if (i < 4) a[i - 2] = rd_a(ws1, 0, i - 2);
          if (i >= 4 && i - 4 < NJ) b0[i - 4] = rd_b(hs1, 0, i - 4);
        }
        if (WS == 2 && i - 2 < LW) issue_W1(k + 2, ws, i - 2);
        if (i - 2 < LH) issue_H1(k + 2, hs, i - 2);
      }
      if (kLive) {
#pragma unroll
        for (int i = 2; i < 8; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, NJ, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          if (i < 4 || i - 4 < NJ) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          if (WS == 2 && i - 2 < LW) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
          if (i - 2 < LH) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      ws = ws1;
      hs = hs1;
      ws2 = ws2 == 2 ? 0 : ws2 + 1;
    }
  };
  const bool live = p0 + wp * kWaveP < M;
  if (live)
    mainloop(std::true_type{});
  else
    mainloop(std::false_type{});
  // loads into LDS still in flight must neither overwrite the exchange below
  // nor outlive the workgroup
  __builtin_amdgcn_s_waitcnt(0);
  barrier_nofence();

  // Statistics of the wave's 128 rows; the lower half's waves take the upper
  // half's through LDS, merge and store.
  float4 st[NJ], dr[NJ];
  auto stats = [&](auto full_tag) {
    constexpr bool kFull = decltype(full_tag)::value;
    const int vbase = v0 + wv * 128;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      float m, s, t;
      int idx;
      column_stats<Lay, kFull>(acc, j, lane, vbase, V, m, idx, s, t);
      st[j] = make_float4(m, s, t, __int_as_float(idx));
      if (kMode == kTarget) {
        float z;
        if (column_target<Lay>(acc, j, lane, vbase, V, col_in[j], z))
          ta.z[p0 + wp * kWaveP + Lay::col(j, lane)] = z;
      }
      if (kMode == kDrawn && __ballot(col_in[j] >= 0)) {
        float best, bz;
        int bidx;
        column_draw<Lay, kFull>(acc, j, lane, vbase, V, col_in[j], sa, best, bidx, bz);
        dr[j] = make_float4(best, __int_as_float(bidx), bz, 0.f);
      }
    }
  };
  if (live) {
    if (v0 + kTileV <= V)
      stats(std::true_type{});
    else
      stats(std::false_type{});
  }
  float4* red = reinterpret_cast<float4*>(smem);  // [kTP] upper half, statistics
  float4* sred = red + kTP;                       // [kTP] upper half, drawn
  if (live && wv == 1 && lane < Lay::kLeaders) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      red[wp * kWaveP + Lay::col(j, lane)] = st[j];
      if (kMode == kDrawn) sred[wp * kWaveP + Lay::col(j, lane)] = dr[j];
    }
  }
  __syncthreads();
  if (live && wv == 0 && lane < Lay::kLeaders) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int c = wp * kWaveP + Lay::col(j, lane), p = p0 + c;
      if (p < M) {
        partials[(size_t)vt * M + p] = merge2(st[j], red[c]);
        if (kMode == kDrawn && col_in[j] >= 0)
          sa.partials[(size_t)vt * M + p] = pick_drawn(dr[j], sred[c]);
      }
    }
  }
#endif
}

}  // namespace
}  // namespace fork
