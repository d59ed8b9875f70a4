// LM-head projection fused with the per-position vocabulary reductions, fp32
// inputs (v_mfma_f32_16x16x4f32).
//
// What bounds it is the fp32 matrix rate: one MFMA of 2048 flop takes 32
// cycles, 1/16 of the bf16 rate, so LDS and L2 traffic are secondary and the
// work goes where it fills the 256 CUs: a workgroup holds 256 vocabulary rows
// x 16 N positions (N = 1, 2, 4, chosen by choose() from the sizes), eight
// waves of 32 rows each, so no matrix work is spent on a padded position tile
// and a small step still spreads over several CUs.  K is staged through LDS in
// 128-byte slabs (32 fp32) by buffer loads that write LDS directly; a wave loads
// its own W rows.  A tile alone on its CU has three slots per operand, so that its
// loads run two stages ahead; with more tiles than CUs two slots (at most 80 KiB)
// let two tiles share a CU, and one's statistics and first loads run under the
// other's main loop.  A 16-byte LDS read gives a
// lane four consecutive K values of a row, the operands of four MFMAs (MFMA m
// sums element m of the four lane groups' chunks).
//
// Each wave takes the statistics of its 32 rows; the eight results of a
// position are merged in order through LDS.  The sums are the same for every
// N, so a row's partials have the same bits whichever tile a launch takes.
#include "lmhead_device.h"
#include "lmhead_tiles.h"

namespace fork {
namespace {

constexpr int kWaves = 8;
constexpr int kWaveRows = 32;

template <int NJ, int kSlots, int kMode>
__device__ __forceinline__ void gemm_f32_body(
    const unsigned char* __restrict__ hidden, const unsigned char* __restrict__ W, int M, int d,
    int V, int nvt, int npt, int pt0, float4* __restrict__ partials,
    const int32_t* __restrict__ rowlist, int Mh, const SampleArgs& sa, const TargetArgs& ta) {
  typedef AccN<NJ, 2> Lay;
  constexpr int kTP = 16 * NJ;  // positions per workgroup
  constexpr int LW = 4;         // W loads of a wave per stage: its own 32 rows
  // hidden loads of a wave per stage; with fewer than eight groups of 8
  // positions several waves load the same group (the same bytes)
  constexpr int kGroups = kTP / 8;
  constexpr int LH = kGroups >= kWaves ? kGroups / kWaves : 1;
  constexpr int kHBytes = kTP * kSlab;
  constexpr int kExchange = kWaves * kTP * 16 * (kMode == kDrawn ? 2 : 1);
  constexpr int kRing = kSlots * (kOperandBytes + kHBytes);
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kRing > kExchange ? kRing : kExchange];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  int vt, pt;
  map_tile(blockIdx.x, nvt * npt, nvt, npt, vt, pt);
  const int v0 = vt * kTileV;
  const int p0 = (pt0 + pt) * kTP;

  const int row_bytes = d * 4;
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

  // A load instruction fills 8 rows x 128 B of LDS (see gemm_narrow.hip).
  const int lrow = lane >> 3;
  auto chunk = [&](int group) { return (lane & 7) ^ lrow ^ (group & 1); };
  auto hgroup = [&](int q) { return kGroups >= kWaves ? wave * LH + q : wave % kGroups; };
  unsigned woff[LW], hoff[LH];
#pragma unroll
  for (int q = 0; q < LW; ++q) {
    const int g = wave * LW + q;
    woff[q] = (unsigned)((g * 8 + lrow) * row_bytes) + (unsigned)(chunk(g) << 4);
  }
#pragma unroll
  for (int q = 0; q < LH; ++q) {
    const int g = hgroup(q), p = g * 8 + lrow;  // p: position within the tile
    int r = p;
    if (listed) {
      r = p0 + p < M ? rowlist[p0 + p] : -1;
      if (r >= Mh) r = -1;
    }
    hoff[q] = r >= 0 ? (unsigned)(r * row_bytes) + (unsigned)(chunk(g) << 4) : kOutOfRange;
  }
  auto at = [&](unsigned off, int s, int group) -> unsigned {
    const bool in = s < kfull || s * 8 + chunk(group) < kchunks;
    return in && off != kOutOfRange ? off + (unsigned)(s * kSlab) : kOutOfRange;
  };
  auto issue = [&](int s, int slot) {
#pragma unroll
    for (int q = 0; q < LW; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsW,
          (__attribute__((address_space(3))) void*)(smem + slot * kOperandBytes +
                                                    (wave * LW + q) * 1024),
          16, at(woff[q], s, wave * LW + q), 0, 0, 0);
#pragma unroll
    for (int q = 0; q < LH; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsH,
          (__attribute__((address_space(3))) void*)(smem + kSlots * kOperandBytes +
                                                    slot * kHBytes + hgroup(q) * 1024),
          16, at(hoff[q], s, hgroup(q)), 0, 0, 0);
  };

  typename Lay::Arr acc;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  const int fr = lane & 15;
  const int kq = lane >> 4;
  const int fx = swz(fr);
  // The given token (kTarget) or draw row (kDrawn) of each column of this lane.
  int col_in[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int p = p0 + Lay::col(j, lane);
    const int32_t* src = kMode == kTarget ? ta.token : sa.row;
    col_in[j] = kMode != kGreedy && p < M ? src[p] : -1;
  }

  constexpr int kAhead = kSlots > 1 ? kSlots - 1 : 1;  // stages issued before their turn
#pragma unroll
  for (int s = 0; s < kAhead; ++s) issue(s, s);
  int slot = 0, next = kAhead;
  for (int k = 0; k < nk; ++k) {
    // stage k resident (with three slots stage k + 1 may be in flight), all
    // waves done with stage k - 1, whose slot takes stage k + kAhead; stages
    // past the end read as zero into slots nobody reads
    wait_vm_lgkm0<(kAhead - 1) * (LW + LH)>();
    barrier_nofence();
    if (kSlots > 1) issue(k + kAhead, next);
    const unsigned char* sw = smem + slot * kOperandBytes + (wave * kWaveRows + fr) * kSlab;
    const unsigned char* sh = smem + kSlots * kOperandBytes + slot * kHBytes + fr * kSlab;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int c = ((2 * kq + kk) ^ fx) << 4;
      f32x4 a[2], b[NJ];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const f32x4*>(sw + 16 * i * kSlab + c);
#pragma unroll
      for (int j = 0; j < NJ; ++j) b[j] = *reinterpret_cast<const f32x4*>(sh + 16 * j * kSlab + c);
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][m], b[j][m], acc[i][j], 0, 0, 0);
    }
    slot = slot == kSlots - 1 ? 0 : slot + 1;
    next = next == kSlots - 1 ? 0 : next + 1;
  }
  // loads into LDS still in flight must neither overwrite the exchange below
  // nor outlive the workgroup
  __builtin_amdgcn_s_waitcnt(0);
  barrier_nofence();

  float4* red = reinterpret_cast<float4*>(smem);  // [kWaves][kTP] statistics
  float4* sred = red + kWaves * kTP;              // [kWaves][kTP] drawn
  auto stats = [&](auto full_tag) {
    constexpr bool kFull = decltype(full_tag)::value;
    const int vbase = v0 + wave * kWaveRows;
    float4 st[NJ];  // all columns before the first is stored: their chains overlap
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      float m, s, t;
      int idx;
      column_stats<Lay, kFull>(acc, j, lane, vbase, V, m, idx, s, t);
      st[j] = make_float4(m, s, t, __int_as_float(idx));
    }
    if (lane < Lay::kLeaders) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) red[wave * kTP + Lay::col(j, lane)] = st[j];
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int c = Lay::col(j, lane);
      if (kMode == kTarget) {
        float z;
        if (column_target<Lay>(acc, j, lane, vbase, V, col_in[j], z)) ta.z[p0 + c] = z;
      }
      if (kMode == kDrawn && __ballot(col_in[j] >= 0)) {
        float best, bz;
        int bidx;
        column_draw<Lay, kFull>(acc, j, lane, vbase, V, col_in[j], sa, best, bidx, bz);
        if (lane < Lay::kLeaders)
          sred[wave * kTP + c] = make_float4(best, __int_as_float(bidx), bz, 0.f);
      }
    }
  };
  if (v0 + kTileV <= V)
    stats(std::true_type{});
  else
    stats(std::false_type{});
  __syncthreads();
  if (tid < kTP && p0 + tid < M) {
    const int p = p0 + tid;
    float4 r = red[tid];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) r = merge2(r, red[w * kTP + tid]);
    partials[(size_t)vt * M + p] = r;
    if (kMode == kDrawn && sa.row[p] >= 0) {
      float4 o = sred[tid];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) o = pick_drawn(o, sred[w * kTP + tid]);
      sa.partials[(size_t)vt * M + p] = o;
    }
  }
}

template <int NJ, int kSlots, int kMode>
__global__ __launch_bounds__(64 * kWaves, kSlots == 1 ? 6 : kSlots == 2 ? 4 : 2) void gemm_f32_kernel(
    const unsigned char* __restrict__ hidden, const unsigned char* __restrict__ W, int M, int d,
    int V, int nvt, int npt, int pt0, float4* __restrict__ partials,
    const int32_t* __restrict__ rowlist, int Mh, SampleArgs sa, TargetArgs ta) {
  gemm_f32_body<NJ, kSlots, kMode>(hidden, W, M, d, V, nvt, npt, pt0, partials, rowlist, Mh, sa, ta);
}

template <int NJ, int kSlots>
hipError_t launch(const void* hidden, const void* W, int M, int d, int V, float4* partials,
                  const int32_t* rowlist, int Mh, const SampleArgs& sample,
                  const TargetArgs& target, hipStream_t stream) {
  const int nvt = num_vocab_tiles(V);
  const int npt = (int)(((long long)M + 16 * NJ - 1) / (16 * NJ));
  const auto* h = static_cast<const unsigned char*>(hidden);
  const auto* w = static_cast<const unsigned char*>(W);
  // a launch holds fewer than 2^32 work-items: more position tiles than that
  // go in further launches
  const int most = (int)(((1LL << 32) - 1) / (64 * kWaves) / nvt);
  for (int pt0 = 0; pt0 < npt; pt0 += most) {
    const int n = npt - pt0 < most ? npt - pt0 : most;
    const dim3 grid((unsigned)(nvt * n)), block(64 * kWaves);
#define FORK_LAUNCH(MODE)                                                                      \
  hipLaunchKernelGGL((gemm_f32_kernel<NJ, kSlots, MODE>), grid, block, 0, stream, h, w, M, d, V, nvt, \
                     n, pt0, partials, rowlist, Mh, sample, target)
    if (target.token)
      FORK_LAUNCH(kTarget);
    else if (sample.row)
      FORK_LAUNCH(kDrawn);
    else
      FORK_LAUNCH(kGreedy);
#undef FORK_LAUNCH
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// 16-position columns per wave: the least time of the launch by the rounds it
// takes.  More than 256 tiles run two to a CU (the two-slot ring), rounds of 512:
// a pair of tiles of 1, 2 or 4 columns takes 1.75, 2.25, 3.8 times one tile of one
// column alone, and tiles alone on their CU (up to 256, the three-slot ring, or the
// rest of the rounds) 1, 1.3, 2.2.  Over 1106 random sizes (d = 4 .. 8192, M to 10000,
// V to 126000) the choice is 0.8% slower than the best of the six for each size and
// 18% at most.  Tiles of 8 columns, one to a CU, were 3 to 20% slower than 4 columns
// two to a CU wherever several rounds run (M = 4000, V = 41661, us per 256 x 64
// tile and CU: d = 128 12.1 / 10.6, 256 19.7 / 18.2, 1024 67.6 / 64.2).
// Rows of one stage (d <= 32) need one slot: three tiles of 4 columns to a CU (4.7
// -> 4.0 us).  A kernel with 256 positions per workgroup and registers between
// global memory and LDS was faster only where a tile is little more than its
// statistics: d <= 32 by up to 8%, d = 40 .. 70 by up to 11% (6.0 to 7.3 us against
// 6.7 to 7.3), d = 70 .. 110 by up to 6%; larger d by 3% at most, and up to 5 times
// slower where few tiles run.
int choose(int M, int V) {
  const long long nvt = num_vocab_tiles(V);
  const int cols[3] = {1, 2, 4};
  const int alone[3] = {100, 130, 220}, pair[3] = {175, 225, 380};
  int best = 0;
  long long least = 0;
  for (int i = 0; i < 3; ++i) {
    const long long tiles = nvt * (((long long)M + 16 * cols[i] - 1) / (16 * cols[i]));
    const long long rest = tiles % (2 * kCus);
    const long long c = tiles / (2 * kCus) * pair[i] +
                        (rest == 0 ? 0 : rest <= kCus ? alone[i] : pair[i]);
    if (i == 0 || c < least) {
      best = i;
      least = c;
    }
  }
  return cols[best];
}

}  // namespace

hipError_t launch_gemm_f32(const void* hidden, const void* W, int M, int d, int V,
                           float4* partials, const int32_t* rowlist, int Mh,
                           const SampleArgs& sample, const TargetArgs& target,
                           hipStream_t stream) {
  const int n = choose(M, V);
  const bool two =
      num_vocab_tiles(V) * (((long long)M + 16 * n - 1) / (16 * n)) > kCus;  // two to a CU
#define FORK_F32(NJ)                                                                              \
  (two ? launch<NJ, 2>(hidden, W, M, d, V, partials, rowlist, Mh, sample, target, stream) \
       : launch<NJ, 3>(hidden, W, M, d, V, partials, rowlist, Mh, sample, target, stream))
  if (n == 1) return FORK_F32(1);
  if (n == 2) return FORK_F32(2);
  // rows of one stage: one slot, 40 KiB, three to a CU
  if (two && d <= kSlab / 4)
    return launch<4, 1>(hidden, W, M, d, V, partials, rowlist, Mh, sample, target, stream);
  return FORK_F32(4);
#undef FORK_F32
}

}  // namespace fork
