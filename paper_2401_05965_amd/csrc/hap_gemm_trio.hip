/*
 * Instances of gemm_trio_kernel (hap_gemm_kernels.h): bf16 operands and output (an fp32 output is a weight gradient's, over long contractions as a rule).
 */
#include "hap_gemm_kernels.h"

namespace hap_gemm_detail {

namespace {

template <typename TC, bool AKC, bool BKC>
int launch(const GemmArgs& a, int groups, hipStream_t st) {
  static bool configured[64] = {};
  return launch_lds_kernel<TC, 128, 128, false>(&gemm_trio_kernel<TC, AKC, BKC>, configured, (size_t)3 * (128 + 128) * 32 * 2, 256, a, groups, st);
}

}  // namespace

int run_trio(const hap_gemm_problem* p, const GemmArgs& a, int groups, hipStream_t st) {
  if (p->a_kcontig && p->b_kcontig) return launch<__bf16, true, true>(a, groups, st);
  if (p->a_kcontig) return launch<__bf16, true, false>(a, groups, st);
  return launch<__bf16, false, false>(a, groups, st);
}

}  // namespace hap_gemm_detail
