// Binary32 instances of the in-place product for any layout (gemm_any.hpp).
#include "gemm_any.hpp"

namespace symt {

hipError_t launch_gemm_any_f32(const AnyLaunch& l, int64_t batch, int M, int N, int K, const void* A, const void* B,
                               void* C, hipStream_t s, const FusedTables* f, void* part, size_t part_bytes) {
  const AnySteps st = any_steps(K, f->any_krun, 32);
  return l.ch == 16
             ? launch_any_typed<float, 16>(l.tile, l.am, l.cb, batch, M, N, st, A, B, C, s, f, part, part_bytes, l.sk)
             : launch_any_typed<float, 4>(l.tile, l.am, l.cb, batch, M, N, st, A, B, C, s, f, part, part_bytes, l.sk);
}

}  // namespace symt
