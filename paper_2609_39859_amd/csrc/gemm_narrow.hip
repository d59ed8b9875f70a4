// LM-head projection fused with the per-position vocabulary reductions, for
// few positions or few tiles (bf16): the kernel of gemm_stats.hip with 64, 128
// or 256 positions per workgroup instead of 256 always.
//
// What bounds these shapes is not the matrix units.  With one or two hundred
// positions and a large vocabulary the step streams W from HBM once; with a
// small vocabulary (a share of a split head, a small model) the 256-position
// tiles leave most of the 256 CUs without work, and a tile's time is its serial
// chain of stages, which grows with the positions it holds: 1 : 1.45 : 1.95
// for 64, 128 and 256 positions at equal K.  So:
//   * a wave holds 128 vocabulary rows x 16 N positions (N = 1, 2, 4), eight
//     waves 2 (vocabulary) x 4 (positions): the loads, stages and fragment
//     layout are those of the 256-position kernel, only the hidden ring and
//     the accumulators shrink with N;
//   * W, read once when all positions share one tile, is loaded with the
//     nontemporal policy if it cannot stay in the 256 MB last-level cache
//     anyway: 6.8 instead of 6.3 TB/s on a load-only kernel of this access
//     pattern.  (A W that fits is better cached: with one 130 MB W read by
//     every step 37 us cached, 51 us nontemporal.)
// Measured, likelihoods of M rows (LM head and merge, us, replayed as a graph),
// 256-position kernel -> this one: d = 4096, V = 126464: M = 32 189 -> 165, 64 231
// -> 203, 128 200 -> 178, 256 250 -> 231; d = 4096: M = 256, V = 15808 79 -> 47, M =
// 128, V = 2000 54 -> 38; M = 128: d = 1024, V = 32000 26 -> 21, d = 256, V = 2000
// 17 -> 10.
// With more than one round of 64-position tiles a two-slot W ring (80 KiB) puts
// two workgroups on a CU, so that one's statistics and first loads run under the
// other's main loop (the same measure, M = 64, V = 83339, d = 224 / 1024 / 4096:
// 20.0 / 39.3 / 151 -> 18.2 / 35.7 / 140; V = 126464, d = 4096, where W streams at
// the read rate, 205 -> 204); with one round the third slot is worth more (M =
// 130, V = 9000, d = 4096: 41 against 58).
// Tried and not kept: 128 vocabulary rows per workgroup with two workgroups
// per CU (equal when W streams, slower otherwise: twice the hidden traffic),
// four W slots instead of three (equal), loads of W and hidden issued by
// different waves (slower), both halves of a tile interleaved per wave with
// hidden fragments kept in registers (equal at 256 positions).
//
// The statistics of a wave's 128 rows and their merge are those of
// gemm_stats.hip, in the same order over the same sums, so partials have the
// same bits whichever kernel a launch takes.
#include "gemm_narrow_body.h"

namespace fork {
namespace {

template <int NJ, bool kNt, int kMode, int WS>
__global__ __launch_bounds__(64 * kWaves, WS == 2 ? 4 : 2) void gemm_narrow_kernel(
    const unsigned char* __restrict__ hidden, const unsigned char* __restrict__ W, int M, int d,
    int V, int nvt, int npt, float4* __restrict__ partials,
    const int32_t* __restrict__ rowlist, int Mh, SampleArgs sa, TargetArgs ta) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[narrow_lds_bytes(NJ, WS)];
  int vt, pt;
  map_tile(blockIdx.x, nvt * npt, nvt, npt, vt, pt);
  gemm_narrow_body<NJ, kNt, kMode, WS>(smem, hidden, W, M, d, V, vt, pt * 64 * NJ, partials,
                                       rowlist, Mh, sa, ta);
}

template <int NJ, bool kNt, int WS>
hipError_t launch(const void* hidden, const void* W, int M, int d, int V, float4* partials,
                  const int32_t* rowlist, int Mh, const SampleArgs& sample,
                  const TargetArgs& target, hipStream_t stream) {
  const int nvt = num_vocab_tiles(V);
  const int npt = (M + 64 * NJ - 1) / (64 * NJ);
  const dim3 grid((unsigned)(nvt * npt)), block(64 * kWaves);
  const auto* h = static_cast<const unsigned char*>(hidden);
  const auto* w = static_cast<const unsigned char*>(W);
#define FORK_LAUNCH(MODE)                                                                        \
  hipLaunchKernelGGL((gemm_narrow_kernel<NJ, kNt, MODE, WS>), grid, block, 0, stream, h, w, M, d, \
                     V, nvt, npt, partials, rowlist, Mh, sample, target)
  if (target.token)
    FORK_LAUNCH(kTarget);
  else if (sample.row)
    FORK_LAUNCH(kDrawn);
  else
    FORK_LAUNCH(kGreedy);
#undef FORK_LAUNCH
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_narrow(int positions, bool nontemporal, bool two_per_cu,
                              const void* hidden, const void* W, int M, int d, int V,
                              float4* partials, const int32_t* rowlist, int Mh, const SampleArgs& sample, const TargetArgs& target,
                              hipStream_t stream) {
#define FORK_NARROW(NJ, NT, WS) \
  launch<NJ, NT, WS>(hidden, W, M, d, V, partials, rowlist, Mh, sample, target, stream)
  if (positions == 64 && two_per_cu)
    return nontemporal ? FORK_NARROW(1, true, 2) : FORK_NARROW(1, false, 2);
  if (positions == 64) return nontemporal ? FORK_NARROW(1, true, 3) : FORK_NARROW(1, false, 3);
  if (positions == 128) return nontemporal ? FORK_NARROW(2, true, 3) : FORK_NARROW(2, false, 3);
  return FORK_NARROW(4, true, 3);
#undef FORK_NARROW
}

}  // namespace fork
