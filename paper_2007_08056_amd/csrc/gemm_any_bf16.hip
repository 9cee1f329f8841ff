// Split-bf16 instances of the in-place product for any layout (gemm_any.hpp).
#include "gemm_any.hpp"

namespace symt {
namespace {

template <int CH, int AM, typename TC>
hipError_t launch_tile(int tile, int64_t batch, int M, int N, const AnySteps& st, const void* A, const void* B, void* C,
                       hipStream_t s, const FusedTables* f, void* part, size_t part_bytes, bool sk) {
  // (128 x 128 with 4-byte loads: their sources and two accumulators exceed the registers)
  if constexpr (CH == 16)
    if (tile == 0)
      return launch_any_kernel<float, 128, 128, 2, 2, CH, AM, false, true, TC>(batch, M, N, st, A, B, C, s, f, part,
                                                                                part_bytes, sk);
  if (tile <= 1)
    return launch_any_kernel<float, 128, 64, 2, 2, CH, AM, false, true, TC>(batch, M, N, st, A, B, C, s, f, part,
                                                                             part_bytes, sk);
  return launch_any_kernel<float, 64, 64, 2, 2, CH, AM, false, true, TC>(batch, M, N, st, A, B, C, s, f, part,
                                                                          part_bytes, sk);
}

template <typename TC>
hipError_t launch_out(const AnyLaunch& l, int64_t batch, int M, int N, const AnySteps& st, const void* A, const void* B,
                      void* C, hipStream_t s, const FusedTables* f, void* part, size_t part_bytes) {
  if (l.ch == 16)
    return l.am == 0 ? launch_tile<16, 0, TC>(l.tile, batch, M, N, st, A, B, C, s, f, part, part_bytes, l.sk)
                     : launch_tile<16, 1, TC>(l.tile, batch, M, N, st, A, B, C, s, f, part, part_bytes, l.sk);
  return l.am == 0 ? launch_tile<4, 0, TC>(l.tile, batch, M, N, st, A, B, C, s, f, part, part_bytes, l.sk)
                   : launch_tile<4, 1, TC>(l.tile, batch, M, N, st, A, B, C, s, f, part, part_bytes, l.sk);
}

}  // namespace

// C: W in its own type (binary32 or binary64), or the aligned W (binary64).
hipError_t launch_gemm_any_bf16x3(const AnyLaunch& l, int64_t batch, int M, int N, int K, const void* A, const void* B,
                                  void* C, hipStream_t s, const FusedTables* f, void* part, size_t part_bytes) {
  const AnySteps st = any_steps(K, f->any_krun, 32);
  return f->rc && f->c_bytes == 4 ? launch_out<float>(l, batch, M, N, st, A, B, C, s, f, part, part_bytes)
                                  : launch_out<double>(l, batch, M, N, st, A, B, C, s, f, part, part_bytes);
}

}  // namespace symt
