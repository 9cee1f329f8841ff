// Binary64 instances of the in-place product for any layout (gemm_any.hpp).
#include "gemm_any.hpp"

namespace symt {

hipError_t launch_gemm_any_f64(const AnyLaunch& l, int64_t batch, int M, int N, int K, const void* A, const void* B,
                               void* C, hipStream_t s, const FusedTables* f, void* part, size_t part_bytes) {
  const AnySteps st = any_steps(K, f->any_krun, 16);
  return l.ch == 16 ? launch_any_typed<double, 16, false>(l, batch, M, N, st, A, B, C, s, f, part, part_bytes)
                    : launch_any_typed<double, 4, false>(l, batch, M, N, st, A, B, C, s, f, part, part_bytes);
}

}  // namespace symt
