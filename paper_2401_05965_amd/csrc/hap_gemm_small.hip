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

template <typename TC>
int layouts(const hap_gemm_problem* p, const GemmArgs& a, int bm, int groups, hipStream_t st) {
  if (p->a_kcontig && p->b_kcontig) return bm == 32 ? launch<TC, true, true, 32>(a, groups, st) : launch<TC, true, true, 64>(a, groups, st);
  if (p->a_kcontig) return bm == 32 ? launch<TC, true, false, 32>(a, groups, st) : launch<TC, true, false, 64>(a, groups, st);
  return launch<TC, false, false, 64>(a, groups, st);       // (an M-contiguous operand's LDS rows are 128 bytes or more)
}

}  // namespace

int run_small(const hap_gemm_problem* p, const GemmArgs& a, int bm, int groups, hipStream_t st) {
  return p->c_dtype == HAP_BF16 ? layouts<__bf16>(p, a, bm, groups, st) : layouts<float>(p, a, bm, groups, st);
}

}  // namespace hap_gemm_detail
