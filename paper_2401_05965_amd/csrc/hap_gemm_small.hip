/*
 * Instances of gemm_small_kernel (hap_gemm_kernels.h): bf16 operands, bf16 or fp32 output.
 */
#include "hap_gemm_kernels.h"

namespace hap_gemm_detail {

namespace {

template <typename TC, bool AKC, bool BKC, int BM>
int launch(const GemmArgs& a, int groups, hipStream_t st) {
  static bool configured[64] = {};
  return launch_lds_kernel<TC, BM, 64, false>(&gemm_small_kernel<TC, AKC, BKC, BM>, configured, (size_t)kSmallLds<BM>, 512, a, groups, st);
}

}  // namespace

/* bf16 outputs from operands of all forms of the path, fp32 outputs (weight gradients, factor rebuilds) from M- / N-contiguous ones; an
 * M-contiguous operand's LDS rows are 128 bytes or more, so its tiles are of 64 rows. */
int run_small(const hap_gemm_problem* p, const GemmArgs& a, int bm, int groups, hipStream_t st) {
  if (p->c_dtype == HAP_F32) return launch<float, false, false, 64>(a, groups, st);
  if (p->a_kcontig && p->b_kcontig) return bm == 32 ? launch<__bf16, true, true, 32>(a, groups, st) : launch<__bf16, true, true, 64>(a, groups, st);
  if (p->a_kcontig) return bm == 32 ? launch<__bf16, true, false, 32>(a, groups, st) : launch<__bf16, true, false, 64>(a, groups, st);
  return launch<__bf16, false, false, 64>(a, groups, st);
}

}  // namespace hap_gemm_detail
