/*
 * Instances of gemm_pp_kernel (hap_gemm_kernels.h): bf16 operands, bf16 or fp32 output.
 */
#include "hap_gemm_kernels.h"

namespace hap_gemm_detail {

namespace {

template <typename TC, bool AKC, bool BKC, int BM, int BN, int WGM, int WGN>
int launch(const GemmArgs& a, int groups, hipStream_t st) {
  constexpr int BK = 32, STAGES = 4;
  static bool configured[64] = {};
  return launch_lds_kernel<TC, BM, BN>(&gemm_pp_kernel<TC, AKC, BKC, BM, BN, BK, WGM, WGN, STAGES>, configured,
                                       (size_t)STAGES * (BM + BN) * BK * 2, 64 * WGM * WGN, a, groups, st);
}

template <typename TC, int BM, int BN, int WGM, int WGN>
int layouts(const hap_gemm_problem* p, const GemmArgs& a, int groups, hipStream_t st) {
  // (both operands K-contiguous: the planner hands that layout to the two-stage kernel)
  if (p->a_kcontig && p->b_kcontig) return hap_fail(HAP_EDEVICE, "internal: no ping-pong kernel for this layout");
  if (p->a_kcontig) return launch<TC, true, false, BM, BN, WGM, WGN>(a, groups, st);
  if (!p->b_kcontig) return launch<TC, false, false, BM, BN, WGM, WGN>(a, groups, st);
  return launch<TC, false, true, BM, BN, WGM, WGN>(a, groups, st);
}

}  // namespace

int run_pp(const hap_gemm_problem* p, const GemmArgs& a, int groups, hipStream_t st) {
  if (p->c_dtype == HAP_BF16) return layouts<__bf16, 256, 256, 2, 4>(p, a, groups, st);
  return layouts<float, 256, 256, 2, 4>(p, a, groups, st);
}

}  // namespace hap_gemm_detail
