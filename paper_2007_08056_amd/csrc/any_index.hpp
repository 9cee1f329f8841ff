// Index arithmetic of the in-place product for any layout (gemm_any.hpp), shared
// by its kernel and the host-side replay that checks it: which element every
// loaded byte of a tile's LDS image is, and where the MFMA operand reads find it.
//
// A tile's layouts (AM): 0 = rows along K ([m][K-step of 128 bytes]), 1 = K-major
// ([k][m]), 2 = K-major complex pairs ([k / 2][m][re, im]).  B is [k][n], or with
// CB (complex V in place) its complex rows [k / 2][n] only.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace symt {

// K-steps of a product: K stepped plainly, or run by run (krun > 0, spr steps per run).
struct AnySteps {
  int K, krun, spr, nk;
};
inline AnySteps any_steps(int K, int krun, int bk) {
  const int spr = krun > 0 ? (krun + bk - 1) / bk : 0;
  return AnySteps{K, krun, spr, krun > 0 ? K / krun * spr : (K + bk - 1) / bk};
}
// Step kt: its first K index and valid depth.
__host__ __device__ inline void any_step(const AnySteps& st, int kt, int bk, int& k0, int& kv) {
  if (st.krun > 0) {
    const int run = kt / st.spr, s = kt - run * st.spr;
    k0 = run * st.krun + s * bk;
    kv = st.krun - s * bk;
  } else {
    k0 = kt * bk;
    kv = st.K - k0;
  }
  if (kv > bk) kv = bk;
}

// 16-byte chunk swizzle of LDS row k of a [k][columns] tile (row bytes ROW), so
// that the rows one fragment read touches (4 of them; 2 of complex rows) fall on
// distinct banks.  A row holds a multiple of 8 chunks and the swizzle stays in it.
// Q4: the fragments of a 32-deep split-bf16 MFMA, whose four lane groups read K
// indices 4 apart (any_k_bf16) instead of neighbours.
template <int ES, int ROW, bool PAIRS, bool Q4 = false>
__host__ __device__ inline int any_swz(int k) {
  static_assert(!Q4 || (ES == 4 && !PAIRS && ROW % 256 == 0), "split-bf16 rows");
  if constexpr (Q4) return ((k >> 2) & 3) << 2;
  else if constexpr (PAIRS) return ROW % 256 == 0 ? (k & 1) << (ES == 8 ? 3 : 2) : 0;
  else if constexpr (ES == 8) return ROW % 256 == 0 ? (k & 1) << 3 : 0;
  else return ROW % 256 == 0 ? (k & 3) << 2 : ((k >> 1) & 1) << 2;
}

// K index (of a 32-deep step) of element j of lane group g's split-bf16 fragment: a
// permutation of the step, the same for A and B, so that a row-major A still reads
// 16-byte chunks (j 0-3 and 4-7) and rows of [k][columns] fall on distinct banks.
__host__ __device__ inline int any_k_bf16(int g, int j) { return 16 * (j >> 2) + 4 * g + (j & 3); }

// The element behind byte p of A's LDS tile: row m and first K index k of the
// step it belongs to (AM = 2: an even k, the pair), and its byte `sub` past the
// start of element (m, 0 of the step) (AM = 0) or of element (m, k) (else).
struct AnySlot {
  int line, k, sub;   // line: m of A, n of B
};
template <int ES, int BM, int AM, bool Q4 = false>
__host__ __device__ inline AnySlot any_a_slot(int p) {
  constexpr int ROW = AM == 0 ? 128 : AM == 1 ? BM * ES : 2 * BM * ES;
  const int r = p / ROW, b = p % ROW;
  if constexpr (AM == 0) {
    const int src = (((b >> 4) ^ ((r >> 1) & 7)) << 4) | (b & 15);
    return AnySlot{r, src / ES, src};
  } else {
    constexpr int PE = AM == 2 ? 2 * ES : ES;
    const int src = (((b >> 4) ^ any_swz<ES, ROW, AM == 2, Q4>(r)) << 4) | (b & 15);
    return AnySlot{src / PE, AM == 2 ? 2 * r : r, src % PE};
  }
}
template <int ES, int BN, bool CB, bool Q4 = false>
__host__ __device__ inline AnySlot any_b_slot(int p) {
  constexpr int ROW = BN * ES;
  const int r = p / ROW, b = p % ROW;
  const int src = (((b >> 4) ^ any_swz<ES, ROW, CB, Q4>(r)) << 4) | (b & 15);
  return AnySlot{src / ES, CB ? 2 * r : r, src % ES};
}

// Byte of A's LDS tile that holds element (m, k) of the step, and of B's that
// holds (k, n) (CB: of V's element, before the sign of the odd real rows).
template <int ES, int BM, int AM, bool Q4 = false>
__host__ __device__ inline int any_a_off(int m, int k) {
  if constexpr (AM == 0) {
    constexpr int VE = 16 / ES;
    return m * 128 + (((k / VE) ^ ((m >> 1) & 7)) << 4) + (k % VE) * ES;
  } else if constexpr (AM == 1) {
    return k * BM * ES + ((((m * ES) >> 4) ^ any_swz<ES, BM * ES, false, Q4>(k)) << 4) + ((m * ES) & 15);
  } else {
    const int kc = k >> 1, mb = m * 2 * ES;
    return kc * 2 * BM * ES + (((mb >> 4) ^ any_swz<ES, 2 * BM * ES, true>(kc)) << 4) + (mb & 15) + (k & 1) * ES;
  }
}
template <int ES, int BN, bool CB, bool Q4 = false>
__host__ __device__ inline int any_b_off(int k, int n) {
  const int r = CB ? k >> 1 : k, nb = (CB ? n ^ (k & 1) : n) * ES;
  return r * BN * ES + (((nb >> 4) ^ any_swz<ES, BN * ES, CB, Q4>(r)) << 4) + (nb & 15);
}

// Lines (rows m of A, columns n of B) past the end are clamped: the last start of
// a lane load of CH bytes over lines of PE bytes each.
template <int CH, int PE>
__host__ __device__ inline int any_last_line(int lines) {
  return lines - (CH == 16 && PE < 16 ? 16 / PE : 1);
}

}  // namespace symt
