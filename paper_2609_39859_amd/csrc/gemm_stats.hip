// LM-head projection fused with the per-position vocabulary reductions.
//
// For every position r (a row of `hidden`) the model's categorical over the
// vocabulary is softmax(z) with z_v = <hidden_r, W_v> (Fork-dLLM paper,
// Section 2, "Sampling in masked dLLMs").  The step needs, per position, the
// greedy candidate, its probability (the confidence c_t^k), its log-
// probability (ForkGRPO's ratio, Section 3.2) and the entropy (Section 3.1).
// All of them follow from four numbers per (position, vocabulary tile) that
// this kernel produces straight from the MFMA accumulators, so the [M, V]
// logits never leave the registers:
//   m   = max_v z_v                 idx = lowest v attaining m
//   s   = sum_v exp(z_v - m)        t   = sum_v exp(z_v - m) * (z_v - m)
//
// This file: the bf16 kernel with 256 positions per workgroup, and the launch
// (the choice of its kernel: lmhead_tiles.h).  Fewer positions per workgroup are in
// gemm_narrow.hip, fp32 inputs in gemm_f32.hip.
//
// Work decomposition (gfx950 / CDNA4):
//   * one workgroup = 256 vocabulary rows x 256 positions, 8 wave64s laid out
//     2 (vocabulary) x 4 (positions); each wave owns 128 x 64 outputs (fp32
//     accumulators): 8 x 4 blocks of 16 x 16 (v_mfma_f32_16x16x32_bf16);
//   * the MFMA "A" operand is W (vocabulary on the MFMA M axis) and "B" is
//     hidden, so each lane's accumulators hold vocabulary values of whole
//     positions: the vocabulary reduction is mostly in-lane (32 values per
//     position), plus shuffles between the lanes holding the same
//     position and one LDS exchange between the two vocabulary waves;
//   * K is staged through LDS in 128-byte slabs per row (whole cache lines),
//     the 16-byte chunk c of row r stored at chunk slot c ^ f(r) with
//     f(r) = (r & 7) ^ ((r >> 3) & 1): the fragment reads of 16 consecutive
//     lanes (16 rows, one chunk) then hit 16 distinct bank groups;
//   * workgroups are renumbered so that each XCD (private L2) walks a
//     contiguous range of tiles, sweeping groups of kGroupV vocabulary
//     stripes across all position tiles, so concurrently running workgroups
//     share W and hidden stripes in L2.
//
// K is fed to LDS by buffer loads that write LDS directly (no register
// staging).  W gets a 3-slot ring (prefetched two
// stages ahead: it streams from HBM), hidden a 2-slot ring (one stage ahead:
// it stays in the last-level cache): 5 x 32 KiB = the whole 160 KiB of LDS.
// One barrier per 64-element K stage, placed after the first MFMAs of the
// stage's second 32-element step so that queued MFMAs cover it; the fragment
// reads of the next step are interleaved with the current MFMAs, and the
// buffer loads of later stages are spread over the stage one at a time so
// that no wave stalls its MFMA stream behind a burst of loads.  The 16x16x32
// MFMA shape moves the same bytes per flop as 32x32x16 and, on gfx950,
// sustains a higher clock under the same power limit.
//
// Drawn candidates (sampling temperature tau > 0, Section 2): for the
// positions the caller marks, the epilogue also keeps the maximiser of the
// Gumbel-perturbed keys z_v / tau - log E_v, where E_v = -log(1 - U_v) is an
// exponential draw built from Philox4x32-10 (Salmon et al., SC'11) at
// counter (v / 4, row, step counter, 0): one generator call serves the four
// consecutive vocabulary entries a lane holds in one accumulator group.
#include "gemm_narrow_body.h"
#include "lmhead_tiles.h"

namespace fork {
namespace {

constexpr int kThreads = 512;

static_assert(kTileV == 256 && kTileP == 256, "tile layout assumes 256 x 256");

// Per-(position, tile) statistics from the accumulators of one wave, combined
// across the two vocabulary waves through LDS, stored to partials.  Drawn
// candidates (kDrawn) go through a second LDS exchange and a second partials
// array (see SampleArgs); the logit of a given token (kTarget) is stored by
// the one lane that holds it.  kFull: the tile's 256 vocabulary rows are all
// < V (every tile but a ragged last one), so no row test is compiled in.
template <class Lay, int kMode, bool kFull>
__device__ __forceinline__ void epilogue_tile(typename Lay::Arr& acc, unsigned char* smem,
                                              int tid, int lane, int wv, int wp, int vt, int v0,
                                              const PosMap& pos, int M, int V,
                                              float4* __restrict__ partials, const SampleArgs& sa,
                                              const TargetArgs& ta, const ColIn<Lay>& ci) {
  constexpr bool kDraw = kMode == kDrawn;
  constexpr bool full = kFull;
  float4* red = reinterpret_cast<float4*>(smem);  // [2][kTileP]
  float4* sred = red + 2 * kTileP;                // [2][kTileP], drawn candidates
  const int vbase = v0 + wv * 128;
  const bool leader = lane < Lay::kLeaders;
  // the draw's row of this thread's position, for the store after the exchange
  const int own_pos = pos(tid < kTileP ? tid : 0);
  const int own_row = (kDraw && tid < kTileP && own_pos < M) ? sa.row[own_pos] : -1;
#pragma unroll
  for (int j = 0; j < Lay::kNJ; ++j) {
    float m, s, t;
    int idx;
    column_stats<Lay, kFull>(acc, j, lane, vbase, V, m, idx, s, t);
    const int col = wp * 64 + Lay::col(j, lane);
    if (leader) red[wv * kTileP + col] = make_float4(m, s, t, __int_as_float(idx));
    if (kMode == kTarget) {
      float z;
      if (column_target<Lay>(acc, j, lane, vbase, V, ci.col[j], z)) ta.z[pos(col)] = z;
    }
    if (kDraw) {
      const int srow = ci.col[j];
      if (__ballot(srow >= 0)) {
        float best, bz;
        int bidx;
        column_draw<Lay, full>(acc, j, lane, vbase, V, srow, sa, best, bidx, bz);
        if (leader) sred[wv * kTileP + col] = make_float4(best, __int_as_float(bidx), bz, 0.f);
      }
    }
  }
  __syncthreads();
  if (tid < kTileP) {
    const int r = own_pos;
    if (r < M) {
      partials[(size_t)vt * M + r] = merge2(red[tid], red[kTileP + tid]);
      if (kDraw && own_row >= 0) {
        sa.partials[(size_t)vt * M + r] = pick_drawn(sred[tid], sred[kTileP + tid]);
      }
    }
  }
}

template <class Lay, int kMode>
__device__ __forceinline__ void epilogue(typename Lay::Arr& acc, unsigned char* smem, int tid,
                                         int lane, int wv, int wp, int vt, int v0, const PosMap& pos, int M,
                                         int V, float4* __restrict__ partials,
                                         const SampleArgs& sa, const TargetArgs& ta,
                                         const ColIn<Lay>& ci) {
  if (v0 + kTileV <= V)
    epilogue_tile<Lay, kMode, true>(acc, smem, tid, lane, wv, wp, vt, v0, pos, M, V, partials, sa,
                                    ta, ci);
  else
    epilogue_tile<Lay, kMode, false>(acc, smem, tid, lane, wv, wp, vt, v0, pos, M, V, partials,
                                     sa, ta, ci);
}

template <int kMode, bool kIlv, bool kTail>
__device__ __forceinline__ void gemm_stats_bf16_body(
    const unsigned char* __restrict__ hidden, const unsigned char* __restrict__ W, int M, int d,
    int V, int nvt, int npt, int nbig, float4* __restrict__ partials,
    const int32_t* __restrict__ rowlist, int Mh, const SampleArgs& sa, const TargetArgs& ta) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the name
  // W ring: slots 0..2; hidden ring: slots 3..4
  __shared__ __attribute__((aligned(1024))) unsigned char smem[5 * kOperandBytes];

  // kTail: workgroups past the first nbig take a quarter of a tile each, 64
  // positions of the tiles from nbig on (see tail_tiles).
  if (kTail && (int)blockIdx.x >= nbig) {
    const int quarter = xcd_order(blockIdx.x - nbig, gridDim.x - nbig);
    int vt, pt;
    tile_of(nbig + (quarter >> 2), nvt, npt, vt, pt);
    const int p0 = pt * kTileP + (quarter & 3) * 64;
    if (p0 < M)
      gemm_narrow_body<1, false, kMode, 3>(smem, hidden, W, M, d, V, vt, p0, partials, rowlist, Mh,
                                        sa, ta);
    return;
  }

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wv = wave & 1;   // vocabulary half: rows wv*128 .. +128
  const int wp = wave >> 1;  // position quarter: cols wp*64 .. +64

  int vt, pt;
  map_tile(blockIdx.x, nbig, nvt, npt, vt, pt);
  const int v0 = vt * kTileV;
  const int p0 = pt * kTileP;
  const PosMap pos{p0, pt, npt, kIlv};

  const int row_bytes = d * 2;
  const int kchunks = row_bytes >> 4;      // 16-byte chunks per row
  const int nk = (kchunks + 7) >> 3;       // 128-byte stages

  // Buffer descriptors rooted at this tile's first rows: rows past the end of
  // W / hidden are outside the record count and read as zero.
  const unsigned recW = (unsigned)(min(kTileV, V - v0) * row_bytes);
  // With a row list, position p of the tile is hidden row rowlist[p0 + p]
  // (outside [0, Mh): no row, reads as zero) and the descriptor spans all Mh
  // rows; interleaved positions (kIlv) span all M rows too.
  const bool whole = rowlist != nullptr || kIlv;
  const unsigned recH = whole ? (unsigned)((rowlist ? Mh : M) * row_bytes)
                              : (unsigned)(min(kTileP, M - p0) * row_bytes);
  const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(W + (size_t)v0 * row_bytes), (short)0, (int)recW, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rsH = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(hidden + (whole ? (size_t)0 : (size_t)p0 * row_bytes)), (short)0, (int)recH,
      kBufferWord3);

  // Each load instruction of a wave writes 1 KiB of LDS = 8 rows x 128 B;
  // lane i fills chunk slot i % 8 of row drow + 8q, so it loads the logical
  // chunk stored there.  Rows drow + 8q with odd q differ in bit 3, which
  // flips bit 0 of the swizzle.
  const int slot_in_row = lane & 7;
  const int drow = wave * 32 + (lane >> 3);
  const int dchunk0 = slot_in_row ^ swz(drow);
  const int dchunk1 = dchunk0 ^ 1;
  const unsigned off0 = (unsigned)(drow * row_bytes) + (unsigned)(dchunk0 << 4);
  const unsigned off1 = (unsigned)(drow * row_bytes) + (unsigned)(dchunk1 << 4);
  const unsigned qstride = (unsigned)(8 * row_bytes);
  unsigned qoff[4], hoff[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    qoff[q] = ((q & 1) ? off1 : off0) + (unsigned)q * qstride;
    hoff[q] = qoff[q];
    if (kIlv)
      hoff[q] = (unsigned)(pos(drow + 8 * q) * row_bytes) +
                (unsigned)(((q & 1) ? dchunk1 : dchunk0) << 4);
    if (rowlist) {
      const int p = p0 + drow + 8 * q;
      const int r = p < M ? rowlist[p] : -1;
      hoff[q] = (r >= 0 && r < Mh)
                    ? (unsigned)(r * row_bytes) + (unsigned)(((q & 1) ? dchunk1 : dchunk0) << 4)
                    : kOutOfRange;
    }
  }
  const int kfull = kchunks >> 3;  // stages whose chunks all lie inside d
  auto src_off = [&](const unsigned (&base)[4], int s, int q) -> unsigned {
    if (s < kfull) return base[q] + (unsigned)(s * kSlab);
    // chunks past d read as zero (the offset lies beyond every record count)
    const int c = (q & 1) ? dchunk1 : dchunk0;
    return (s * 8 + c < kchunks) ? base[q] + (unsigned)(s * kSlab) : kOutOfRange;
  };
  auto issue_W1 = [&](int s, int slot, int q) {  // sub-block q of W stage s
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rsW, (__attribute__((address_space(3))) void*)(smem + slot * kOperandBytes + (wave * 4 + q) * 1024),
        16, src_off(qoff, s, q), 0, 0, 0);
  };
  auto issue_H1 = [&](int s, int slot, int q) {  // sub-block q of hidden stage s
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rsH, (__attribute__((address_space(3))) void*)(smem + (3 + slot) * kOperandBytes + (wave * 4 + q) * 1024),
        16, src_off(hoff, s, q), 0, 0, 0);
  };
  auto issue_W = [&](int s, int slot) {
#pragma unroll
    for (int q = 0; q < 4; ++q) issue_W1(s, slot, q);
  };
  auto issue_H = [&](int s, int slot) {
#pragma unroll
    for (int q = 0; q < 4; ++q) issue_H1(s, slot, q);
  };

  Acc16::Arr acc;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // Fragments of one 32-element K step: A fragment i = W rows arow + 16 i,
  // B fragment j = positions brow + 16 j.  Step kk of a stage takes the
  // stage's 16-byte chunks kk, kk + 2, kk + 4, kk + 6: lane group kq =
  // lane / 16 supplies chunk 2 kq + kk of both operands, so each MFMA sums
  // over the step's 32 K values and the two steps cover the stage.  With the
  // swizzle above, this assignment reads LDS without bank conflicts (four
  // consecutive chunks per step do not).  Rows 16 apart share a swizzle.
  const int arow = wv * 128 + (lane & 15);
  const int brow = wp * 64 + (lane & 15);
  const int kq = lane >> 4;
  const int fa = swz(arow), fb = swz(brow);
  auto rd_a = [&](int ws, int kk, int i) {
    const int chunk = 2 * kq + kk;
    return *reinterpret_cast<const bf16x8*>(smem + ws * kOperandBytes + (arow + 16 * i) * kSlab +
                                            ((chunk ^ fa) << 4));
  };
  auto rd_b = [&](int hs, int kk, int j) {
    const int chunk = 2 * kq + kk;
    return *reinterpret_cast<const bf16x8*>(smem + (3 + hs) * kOperandBytes +
                                            (brow + 16 * j) * kSlab + ((chunk ^ fb) << 4));
  };
  // One K step: 32 MFMAs on (a, bc), block row i at a time.  After the four
  // MFMAs of row i, a[i] is refilled with the fragment of step kkn (slots
  // wsn / hsn), and the four bn are read in between.  `dma` spreads four
  // buffer loads over the rows: 1 = W stage s_dma (rows 0..3), 2 = hidden
  // stage s_dma (rows 2..5, after the barrier), into slot slot_dma.
  // kSync >= 0: the stage barrier (with its wait for the next stage's data)
  // comes after the MFMAs of rows 0..kSync, so that queued MFMAs cover it;
  // every read of the step follows the barrier.
  // kLive: the wave's 64 positions include one below M.  A wave whose
  // positions all lie past M (a last position tile with fewer than 256
  // positions) issues no MFMAs and reads no fragments; it still loads its
  // share of every stage and takes every barrier.
  auto step = [&](auto live_tag, auto sync_tag, bf16x8 (&a)[8], const bf16x8 (&bc)[4],
                  bf16x8 (&bn)[4], int wsn, int hsn, int kkn, int dma, int s_dma, int slot_dma) {
    constexpr bool kLive = decltype(live_tag)::value;
    constexpr int kSync = decltype(sync_tag)::value;
    // Reads held back by the barrier (kSync >= 0), in this order: a[0..kSync],
    // then bn[0..3]; row kSync + 1 + r takes item r after its second MFMA
    // and, for r < kExtra, item kRows + r after its fourth.
    constexpr int kRows = 7 - kSync;
    constexpr int kItems = kSync + 5;
    constexpr int kExtra = kItems - kRows > 0 ? kItems - kRows : 0;
    auto held = [&](int item) {
      if (item <= kSync) a[item] = rd_a(wsn, kkn, item);
      else bn[item - kSync - 1] = rd_b(hsn, kkn, item - kSync - 1);
    };
    auto row = [&](int i) {
      const int r = i - kSync - 1;
      if (kLive) {
        acc[i][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], bc[0], acc[i][0], 0, 0, 0);
        acc[i][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], bc[1], acc[i][1], 0, 0, 0);
        if (kSync < 0) {
          if (i < 4) bn[i] = rd_b(hsn, kkn, i);
        } else if (r >= 0 && r < kItems) {
          held(r);
        }
        acc[i][2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], bc[2], acc[i][2], 0, 0, 0);
        acc[i][3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], bc[3], acc[i][3], 0, 0, 0);
        if (kSync < 0 || r >= 0) a[i] = rd_a(wsn, kkn, i);
        if (kSync >= 0 && r >= 0 && r < kExtra) held(kRows + r);
      }
      if (dma == 1 && i < 4) issue_W1(s_dma, slot_dma, i);
      if (dma == 2 && i >= 2 && i < 6) issue_H1(s_dma, slot_dma, i - 2);
    };
    auto order = [&](int i) {
      const int r = i - kSync - 1;
      const bool r1 = kSync < 0 ? i < 4 : (r >= 0 && r < kItems);
      const int n2 = (kSync < 0 || r >= 0 ? 1 : 0) + (kSync >= 0 && r >= 0 && r < kExtra ? 1 : 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // MFMA
      if (r1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // LDS read
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      if (n2 >= 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (n2 >= 2) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if ((dma == 1 && i < 4) || (dma == 2 && i >= 2 && i < 6))
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // buffer load
    };
    if (kSync >= 0) {
#pragma unroll
      for (int i = 0; i <= kSync; ++i) row(i);
#pragma unroll
      for (int i = 0; i <= kSync; ++i)
        if (kLive) order(i);
      __builtin_amdgcn_sched_barrier(0);
      // the next stage's hidden and W resident; all reads of this stage returned
      wait_vm_lgkm0<4>();
      barrier_nofence();
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = kSync + 1; i < 8; ++i) row(i);
#pragma unroll
    for (int i = kSync + 1; i < 8; ++i)
      if (kLive) order(i);
  };
  using NoSync = std::integral_constant<int, -1>;
  using SyncAfterRow1 = std::integral_constant<int, 1>;

  ColIn<Acc16> ci;
  auto mainloop = [&](auto live_tag) {
  constexpr bool kLive = decltype(live_tag)::value;
  bf16x8 a[8], b0[4], b1[4];
  // Load order: H0 W0 W1 H1, then per stage k: W(k+2) during the stage's
  // first K step, H(k+2) during its second, after the stage's barrier (which
  // follows the second step's first eight MFMAs).
  // At the barrier of stage k only W(k+2), the 4 newest loads, may be in
  // flight, and every slot refilled after it belongs to a stage all waves
  // have finished reading.  Stages past the end read as zero into slots
  // nobody reads again.
  issue_H(0, 0);
  issue_W(0, 0);
  issue_W(1, 1);
  issue_H(1, 1);
  wait_vm_lgkm0<8>();  // H0 and W0 resident
  barrier_nofence();
  if (kLive) {
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = rd_a(0, 0, i);
#pragma unroll
    for (int j = 0; j < 4; ++j) b0[j] = rd_b(0, 0, j);
  }
  int ws = 0, hs = 0, ws2 = 2;  // W slots of stages k and k + 2, hidden slot of k
  for (int k = 0; k + 1 < nk; ++k) {
    const int ws1 = ws == 2 ? 0 : ws + 1, hs1 = hs ^ 1;
    step(live_tag, NoSync{}, a, b0, b1, ws, hs, 1, 1, k + 2, ws2);
    __builtin_amdgcn_sched_barrier(0);
    step(live_tag, SyncAfterRow1{}, a, b1, b0, ws1, hs1, 0, 2, k + 2, hs);
    __builtin_amdgcn_sched_barrier(0);
    ws = ws1;
    hs = hs1;
    ws2 = ws2 == 2 ? 0 : ws2 + 1;
  }
  load_col_inputs<Acc16, kMode>(ci, tid, lane, wp, pos, M, sa, ta);
  step(live_tag, NoSync{}, a, b0, b1, ws, hs, 1, 0, 0, 0);
  if (kLive) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b1[j], acc[i][j], 0, 0, 0);
  }
  };
  if (pos(wp * 64) < M)
    mainloop(std::true_type{});
  else
    mainloop(std::false_type{});
  __builtin_amdgcn_s_waitcnt(0);
  barrier_nofence();

  epilogue<Acc16, kMode>(acc, smem, tid, lane, wv, wp, vt, v0, pos, M, V, partials, sa, ta, ci);
#endif
}

// Entry points: positions = hidden rows 0..M-1, or gathered through a row
// list; greedy candidates only, drawn candidates as well, or the logits of
// given tokens.  Separate symbols keep the row-list, drawing and target code
// out of the dense greedy kernel and the variants apart in kernel traces.
#define FORK_GEMM_ARGS                                                                         \
  const unsigned char *__restrict__ hidden, const unsigned char *__restrict__ W, int M, int d, \
      int V, int nvt, int npt, int nbig, float4 *__restrict__ partials
#define FORK_GEMM_ENTRIES(T)                                                                   \
  template <bool kTail>                                                                        \
  __global__ __launch_bounds__(kThreads) void gemm_stats_##T##_kernel(FORK_GEMM_ARGS) {       \
    gemm_stats_##T##_body<kGreedy, false, kTail>(hidden, W, M, d, V, nvt, npt, nbig, partials, nullptr, M,         \
                                   SampleArgs{}, TargetArgs{});                                \
  }                                                                                            \
  template <bool kTail>                                                                        \
  __global__ __launch_bounds__(kThreads) void gemm_stats_##T##_rows_kernel(                   \
      FORK_GEMM_ARGS, const int32_t* __restrict__ rowlist, int Mh) {                           \
    gemm_stats_##T##_body<kGreedy, false, kTail>(hidden, W, M, d, V, nvt, npt, nbig, partials, rowlist, Mh,        \
                                   SampleArgs{}, TargetArgs{});                                \
  }                                                                                            \
  template <bool kTail>                                                                        \
  __global__ __launch_bounds__(kThreads) void gemm_stats_##T##_draw_kernel(FORK_GEMM_ARGS,    \
                                                                          SampleArgs sa) {     \
    gemm_stats_##T##_body<kDrawn, false, kTail>(hidden, W, M, d, V, nvt, npt, nbig, partials, nullptr, M, sa,      \
                                  TargetArgs{});                                               \
  }                                                                                            \
  template <bool kTail>                                                                        \
  __global__ __launch_bounds__(kThreads) void gemm_stats_##T##_rows_draw_kernel(              \
      FORK_GEMM_ARGS, const int32_t* __restrict__ rowlist, int Mh, SampleArgs sa) {            \
    gemm_stats_##T##_body<kDrawn, false, kTail>(hidden, W, M, d, V, nvt, npt, nbig, partials, rowlist, Mh, sa,     \
                                  TargetArgs{});                                               \
  }                                                                                            \
  template <bool kTail>                                                                        \
  __global__ __launch_bounds__(kThreads) void gemm_stats_##T##_target_kernel(FORK_GEMM_ARGS,  \
                                                                            TargetArgs ta) {   \
    gemm_stats_##T##_body<kTarget, false, kTail>(hidden, W, M, d, V, nvt, npt, nbig, partials, nullptr, M,         \
                                   SampleArgs{}, ta);                                          \
  }                                                                                            \
  template <bool kTail>                                                                        \
  __global__ __launch_bounds__(kThreads) void gemm_stats_##T##_rows_target_kernel(            \
      FORK_GEMM_ARGS, const int32_t* __restrict__ rowlist, int Mh, TargetArgs ta) {            \
    gemm_stats_##T##_body<kTarget, false, kTail>(hidden, W, M, d, V, nvt, npt, nbig, partials, rowlist, Mh,        \
                                   SampleArgs{}, ta);                                          \
  }
FORK_GEMM_ENTRIES(bf16)
// Drawing over all rows with interleaved positions (M = 256 * npt).
__global__ __launch_bounds__(kThreads) void gemm_stats_bf16_draw_ilv_kernel(FORK_GEMM_ARGS,
                                                                           SampleArgs sa) {
  gemm_stats_bf16_body<kDrawn, true, false>(hidden, W, M, d, V, nvt, npt, nbig, partials, nullptr, M, sa,
                                     TargetArgs{});
}
#undef FORK_GEMM_ARGS
#undef FORK_GEMM_ENTRIES

}  // namespace

hipError_t launch_gemm_stats(const void* hidden, const void* W, bool bf16, int M, int d, int V,
                             float4* partials, const int32_t* rowlist, int Mh,
                             const SampleArgs& sample, const TargetArgs& target,
                             hipStream_t stream) {
  if (!bf16)
    return launch_gemm_f32(hidden, W, M, d, V, partials, rowlist, Mh, sample, target, stream);
  const TileChoice t = choose_tile(M, d, num_vocab_tiles(V), whole_lines(W, d), 2LL * V * d);
  if (t.narrow)
    return launch_gemm_narrow(t.positions, t.nontemporal, t.two_per_cu, hidden, W, M, d, V, partials,
                              rowlist, Mh, sample, target, stream);
  const int nvt = num_vocab_tiles(V);
  const int npt = num_pos_tiles(M);
  const bool draw = sample.row != nullptr;
  const bool tgt = target.token != nullptr;
  const bool ilv = draw && !rowlist && npt > 1 && M == npt * kTileP &&
                   (long long)M * d * 2 < (1LL << 31);
  const int tail = ilv ? 0 : tail_tiles((long long)nvt * npt);
  const int nbig = nvt * npt - tail;
  const dim3 grid((unsigned)(nbig + 4 * tail)), block(kThreads);
  const auto* h = static_cast<const unsigned char*>(hidden);
  const auto* w = static_cast<const unsigned char*>(W);
#define FORK_LAUNCH1(K, ...) hipLaunchKernelGGL((K), grid, block, 0, stream, h, w, M, d, V, nvt, npt, \
                                                nbig, partials, ##__VA_ARGS__)
#define FORK_LAUNCH(K, ...)                     \
  do {                                          \
    if (tail)                                   \
      FORK_LAUNCH1(K<true>, ##__VA_ARGS__);     \
    else                                        \
      FORK_LAUNCH1(K<false>, ##__VA_ARGS__);    \
  } while (0)
  if (rowlist && tgt)
    FORK_LAUNCH(gemm_stats_bf16_rows_target_kernel, rowlist, Mh, target);
  else if (tgt)
    FORK_LAUNCH(gemm_stats_bf16_target_kernel, target);
  else if (rowlist && draw)
    FORK_LAUNCH(gemm_stats_bf16_rows_draw_kernel, rowlist, Mh, sample);
  else if (ilv)
    FORK_LAUNCH1(gemm_stats_bf16_draw_ilv_kernel, sample);
  else if (rowlist)
    FORK_LAUNCH(gemm_stats_bf16_rows_kernel, rowlist, Mh);
  else if (draw)
    FORK_LAUNCH(gemm_stats_bf16_draw_kernel, sample);
  else
    FORK_LAUNCH(gemm_stats_bf16_kernel);
#undef FORK_LAUNCH
#undef FORK_LAUNCH1
  return hipGetLastError();
}

}  // namespace fork
