/*
 * Instances of gemm_dma_kernel and gemm_kpair_kernel (hap_gemm_kernels.h): bf16 operands, bf16 or fp32 output.
 */
#include "hap_gemm_kernels.h"

namespace hap_gemm_detail {

namespace {

template <typename TC, bool AKC, bool BKC, int BM, int BN, int WGM, int WGN>
int launch(const GemmArgs& a, int groups, hipStream_t st) {
  constexpr int BK = 64, STAGES = 2;
  static bool configured[64] = {};
  return launch_lds_kernel<TC, BM, BN>(&gemm_dma_kernel<TC, AKC, BKC, BM, BN, BK, WGM, WGN, STAGES>, configured,
                                       (size_t)STAGES * (BM + BN) * BK * 2, 64 * WGM * WGN, a, groups, st);
}

template <typename TC, bool AKC, bool BKC>
int launch_kpair(const GemmArgs& a, int groups, hipStream_t st) {
  static bool configured[64] = {};
  return launch_lds_kernel<TC, 128, 128>(&gemm_kpair_kernel<TC, AKC, BKC>, configured, (size_t)2 * 2 * (128 + 128) * 64 * 2, 512, a, groups, st);
}

template <typename TC>
int tiles(const hap_gemm_problem* p, const GemmArgs& a, int tile, int groups, hipStream_t st) {
  if (a.kpair) {
    if (p->a_kcontig && p->b_kcontig) return launch_kpair<TC, true, true>(a, groups, st);
    if (p->a_kcontig) return launch_kpair<TC, true, false>(a, groups, st);
    return launch_kpair<TC, false, false>(a, groups, st);     // (an M-contiguous A with a K-contiguous B is never paired)
  }
  if (tile == 128) {
    if (p->a_kcontig && p->b_kcontig) return launch<TC, true, true, 128, 128, 2, 2>(a, groups, st);
    if (p->a_kcontig) return launch<TC, true, false, 128, 128, 2, 2>(a, groups, st);
    if (!p->b_kcontig) return launch<TC, false, false, 128, 128, 2, 2>(a, groups, st);
    return launch<TC, false, true, 128, 128, 2, 2>(a, groups, st);
  }
  // 256-tiles outside the ping-pong kernel: both operands K-contiguous, or a short contraction (A M-contiguous with B
  // K-contiguous always takes the ping-pong kernel, so that layout of the two-stage kernel is not built at this size)
  if (p->a_kcontig && p->b_kcontig) return launch<TC, true, true, 256, 256, 2, 4>(a, groups, st);
  if (p->a_kcontig) return launch<TC, true, false, 256, 256, 2, 4>(a, groups, st);
  if (!p->b_kcontig) return launch<TC, false, false, 256, 256, 2, 4>(a, groups, st);
  return hap_fail(HAP_EDEVICE, "internal: no 256-tile two-stage kernel for this layout");
}

}  // namespace

int run_dma(const hap_gemm_problem* p, const GemmArgs& a, int tile, int groups, hipStream_t st) {
  return p->c_dtype == HAP_BF16 ? tiles<__bf16>(p, a, tile, groups, st) : tiles<float>(p, a, tile, groups, st);
}

}  // namespace hap_gemm_detail
