// Row-streaming sector product for short contractions (Alg. 2's product step
// where K and N are both at most 64): C[Q] = A[Q] B[Q] with A[Q] tall (M rows),
// f64 or f32.
//
// Such a product moves 8 (K + N) bytes per row of A and C for 2 K N flops, so
// it is bound by HBM (about 6 flops per byte at K = N = 48), not by the matrix
// cores.  This kernel therefore reads every element of A exactly once, straight
// from global memory into the MFMA operand registers (no LDS staging of A),
// keeps all of B[Q] in LDS for the workgroup's lifetime, and writes C straight
// from the accumulators.  Each wave owns blocks of 16 (binary64) or 32 (binary32) rows by all N columns and
// issues the loads of a whole block (K / 4 per 16-row group) before its first
// MFMA, and the next block's loads before this block's MFMAs (table reads run
// further ahead); waves run their row blocks independently (one barrier, after
// B is in LDS).
//
// Operands are addressed through separable offset tables, so the same kernel
// reads A from U's standard form (row offsets ra, column offsets ca, any
// layout of U's modes), B from V's (rb, cb) and writes C into W's (rc, cc);
// a null table stands for the aligned row-major form.  K is summed four
// indices per MFMA (v_mfma_f64_16x16x4_f64, v_mfma_f32_16x16x4_f32): in order in
// binary64, in a fixed order within groups of 16 in binary32 (see below).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "gemm_common.hpp"
#include "plan.hpp"

namespace symt {

namespace {

template <typename T>
struct RowMfma;
// Accumulator rows (lane l, item r; column l % 16): f64 l/16 + 4r, f32 4(l/16) + r.
template <>
struct RowMfma<double> {
  using Acc = d4;
  static __device__ __forceinline__ Acc run(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <>
struct RowMfma<float> {
  using Acc = f4;
  static __device__ __forceinline__ Acc run(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

constexpr int kRowWaves = 4;     // waves per workgroup

// Element strides of the operands that have no tables: A at q aq + m ar + k ac, B at
// q bq + k br + n bc, C at q cq + m cr + n cc.
struct RowStrides {
  int64_t aq, ar, ac, bq, br, bc, cq, cr, cc;
};

// 16-row groups per wave block: one for binary64 (its A, accumulators and
// prefetched A fill two thirds of the registers already), two for binary32
// (each B value read from LDS then feeds two MFMAs)
template <typename T, int KS, int TN>
constexpr int row_groups() {
  return sizeof(T) == 8 ? 1 : 2;
}

// KS: K-steps of 4 (K <= 4 KS); TN: 16-column tiles (N <= 16 TN).
// Grid: (workgroups per Q, Q).  Wave w of workgroup x walks row blocks
// x * kRowWaves + w, stepping by gridDim.x * kRowWaves.
// TR: the MFMA computes the transposed tile (B^T A^T), so that each lane's
// accumulators hold one row of C and a store instruction writes 16 consecutive
// rows (for a W whose rows, not columns, are its contiguous index).
// RV > 1 (A's rows contiguous in aligned runs of RV, as where U's output modes
// trail: A read K-major): lane r of a 16 x RV-row group loads rows RV r ..
// RV r + RV - 1 of one K index with one 16-byte load and feeds them to RV
// MFMAs, whose output row p then stands for row RV p + t of the group.
// Binary32 steps through K in groups of 16: K-step 4 u + t takes index
// 16 u + 4 kq + t at lane group kq (the same sums as 4 s + kq, permuted within
// each group, in every variant); KV = 4 (A's K index contiguous in aligned
// runs of 4): lane (r, kq) loads the four indices 16 u + 4 kq .. + 3 of its row
// with one 16-byte load for K-steps 4 u .. 4 u + 3.
template <typename T, int KS, int TN, bool TR, int RV = 1, int KV = 1>
__global__ __launch_bounds__(64 * kRowWaves, (RV > 1 ? 2 : 1)) void k_gemm_rows(
    const T* __restrict__ A, const T* __restrict__ B, T* __restrict__ C, int M, int N, int K,
    const int64_t* __restrict__ ra, const int64_t* __restrict__ ca, const int64_t* __restrict__ rb,
    const int64_t* __restrict__ cb, const int64_t* __restrict__ rc, const int64_t* __restrict__ cc,
    const RowStrides st) {
  using Acc = typename RowMfma<T>::Acc;
  static_assert(RV == 1 || (!TR && RV * sizeof(T) == 16), "row vectors: 16 bytes, lanes along columns");
  constexpr int kRowGroups = RV > 1 ? 1 : row_groups<T, KS, TN>();
  constexpr int NG = kRowGroups * RV;            // 16-row MFMA groups per block
  constexpr int KP = 4 * KS;
  constexpr int NP = 16 * TN;
  // B rows padded so that the four k-rows of one operand read start 16 * sizeof(T)
  // bytes apart modulo the 256-byte bank cycle
  constexpr int ROWB = NP * static_cast<int>(sizeof(T));
  constexpr int SHIFT = 16 * static_cast<int>(sizeof(T));
  constexpr int PADB = ((SHIFT - ROWB % 256 + 256) % 256) / static_cast<int>(sizeof(T));
  __shared__ T Bs[KP][NP + PADB];
  __shared__ int64_t cols_a[KP];

  const int64_t q = blockIdx.y;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // B[Q] (zero past K and N) and A's column offsets (past K: never read)
  for (int e = tid; e < KP * NP; e += 64 * kRowWaves) {
    const int k = e / NP, n = e - (e / NP) * NP;
    T x = T(0);
    if (k < K && n < N)
      x = B[rb ? rb[q * K + k] + cb[q * N + n] : q * st.bq + k * st.br + n * st.bc];
    Bs[k][n] = x;
  }
  for (int k = tid; k < KP; k += 64 * kRowWaves)
    cols_a[k] = k < K ? (ca ? ca[q * K + k] : k * st.ac) : 0;
  __syncthreads();

  // this lane's output columns: one per 16-column tile, or (TR) four per tile
  constexpr int NC = TR ? 4 : 1;
  int64_t ccol[TN][NC];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < NC; ++r) {
      const int col = j * 16 + (TR ? RowMfma<T>::row(lane, r) : (lane & 15));
      ccol[j][r] = col < N ? (cc ? cc[q * N + col] : col * st.cc) : -1;
    }
  const int kq = lane >> 4;                      // k index within each K-step
  const int64_t blocks = (M + 16 * NG - 1) / (16 * NG);
  const int64_t step = static_cast<int64_t>(gridDim.x) * kRowWaves;
  // Row offsets of block b's A rows (this lane's row of each 16-row group) and
  // of its C rows (this lane's accumulator rows; -1 past M).
  auto a_rows = [&](int64_t b, int64_t (&rbase)[kRowGroups]) {
#pragma unroll
    for (int i = 0; i < kRowGroups; ++i) {
      const int m = min(static_cast<int>(b * 16 * NG) + i * 16 * RV + RV * (lane & 15), M - RV);
      rbase[i] = ra ? ra[q * M + m] : q * st.aq + m * st.ar;
    }
  };
  constexpr int NR = TR ? 1 : 4;                 // C rows per lane and row group
  auto c_rows = [&](int64_t b, int64_t (&crow)[NG][NR]) {
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int i = g / RV, t = g % RV;
        const int row = static_cast<int>(b * 16 * NG) + i * 16 * RV +
                        (TR ? (lane & 15) : RV * RowMfma<T>::row(lane, r) + t);
        crow[g][r] = row < M ? (rc ? rc[q * M + row] : q * st.cq + row * st.cr) : -1;
      }
  };
  // A: lane (r, kq) of group i holds A[m0 + 16 RV i + RV r + t][4 s + kq], t < RV, for every step s
  static_assert(KV == 1 || (RV == 1 && KV * sizeof(T) == 16 && KS % KV == 0), "K vectors: 16 bytes");
  // K index of (step s, lane group kq): binary64 4 s + kq; binary32 16 (s / 4) + 4 kq + s % 4
  constexpr int KO = sizeof(T) == 4 ? 4 : 1;
  static_assert(KS % KO == 0, "whole groups of K-steps");
  auto kidx = [&](int s) { return KO > 1 ? 4 * KO * (s / KO) + KO * kq + s % KO : 4 * s + kq; };
  using AV = VecT<T, RV>;
  auto load_a = [&](const int64_t (&rbase)[kRowGroups], AV (&a)[kRowGroups][KS]) {
#pragma unroll
    for (int i = 0; i < kRowGroups; ++i) {
      if constexpr (KV > 1) {
#pragma unroll
        for (int u = 0; u < KS / KV; ++u) {
          const int k = kidx(KV * u);
          VecT<T, KV> x;
          if (k < K) {
            x = *reinterpret_cast<const VecT<T, KV>*>(A + rbase[i] + cols_a[k]);
          } else {
#pragma unroll
            for (int t = 0; t < KV; ++t) x.v[t] = T(0);
          }
#pragma unroll
          for (int t = 0; t < KV; ++t) a[i][KV * u + t].v[0] = x.v[t];
        }
      } else {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          const int k = kidx(s);
          if (k < K) {
            a[i][s] = *reinterpret_cast<const AV*>(A + rbase[i] + cols_a[k]);
          } else {
#pragma unroll
            for (int t = 0; t < RV; ++t) a[i][s].v[t] = T(0);
          }
        }
      }
    }
  };
  int64_t blk = static_cast<int64_t>(blockIdx.x) * kRowWaves + wave;
  if (blk >= blocks) return;
  // Loads run ahead: A one block ahead, its row offsets two blocks ahead, and
  // each block's C row offsets before its products, so no table read waits on
  // the critical path (the loads complete in issue order).
  AV a[kRowGroups][KS], an[kRowGroups][KS];
  int64_t r1[kRowGroups], r2[kRowGroups];
  a_rows(blk, r1);
  load_a(r1, a);
  if (blk + step < blocks) a_rows(blk + step, r1);
  for (; blk < blocks; blk += step) {
    int64_t crow[NG][NR];
    c_rows(blk, crow);
    const bool more = blk + step < blocks;
    if (blk + 2 * step < blocks) a_rows(blk + 2 * step, r2);
    if (more) load_a(r1, an);
    Acc acc[NG][TN];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[g][j] = Acc{};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const T b = Bs[kidx(s)][j * 16 + (lane & 15)];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const T av = a[g / RV][s].v[g % RV];
          acc[g][j] = TR ? RowMfma<T>::run(b, av, acc[g][j]) : RowMfma<T>::run(av, b, acc[g][j]);
        }
      }
    }
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t cr = crow[g][TR ? 0 : r];
        if (cr < 0) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int64_t cc_ = ccol[j][TR ? r : 0];
          if (cc_ >= 0) C[cr + cc_] = acc[g][j][r];
        }
      }
    if (more) {
#pragma unroll
      for (int i = 0; i < kRowGroups; ++i) {
#pragma unroll
        for (int s = 0; s < KS; ++s) a[i][s] = an[i][s];
        r1[i] = r2[i];
      }
    }
  }
}

// Row-run variant of the transposed tile, where the rows are the contiguous index of
// both A and C: runs of `run` rows (M a multiple of it) at any element alignment, as
// where a small matrix multiplies one mode of a large tensor (the rows are then the
// tensor's trailing modes: 57^3 of them in the (1, 3, 1) pattern of 57-blocks, an odd
// run that no aligned 16-byte access fits).
// What bounds it: HBM, one read of A and one write of C.  A lane loads 16 bytes of
// consecutive rows of one K index (RV rows: 256 bytes per 16 lanes, four K indices
// per load; a row-by-row lane moves a quarter of that per instruction in binary32)
// and RV MFMAs take one row each, output column p of MFMA t standing for row
// RV p + t, so a lane also holds RV consecutive rows of C per column and stores 16
// bytes.  Element-aligned 16-byte accesses are plain global loads and stores on this
// device.  A block of rows never straddles two runs; a run's last block guards each
// element.  One table entry of A and C per block (wave-uniform).  Same K order as
// k_gemm_rows: same bits.  Two or three waves per SIMD rather than the next block's
// loads in registers: a block's A and accumulators take 128 registers at K = N = 64,
// and one wave's products cover the others' loads.
// Measured: 4 x (57 x 57 x 2963088) f32 2555 -> 1716 us (5.4 GB), f64 4105 -> 3450 us;
// 4 x (32 x 32 x 524288) f32 255 -> 111 us (4.9 TB/s), f64 415 -> 209 us.
template <typename T, int KS, int TN>
constexpr int row_run_waves() {
  return (sizeof(T) == 8 ? KS >= 12 : KS == 16) && TN >= 3 ? 2 : 3;   // (three would spill)
}
template <typename T, int V>
struct __attribute__((packed, aligned(sizeof(T)))) RowVec {
  T v[V];
};

// WHOLE: runs of whole 128-byte lines.
template <typename T, int KS, int TN, bool WHOLE>
__global__ __launch_bounds__(64 * kRowWaves, (row_run_waves<T, KS, TN>())) void k_gemm_row_runs(
    const T* __restrict__ A, const T* __restrict__ B, T* __restrict__ C, int M, int N, int K,
    const int64_t* __restrict__ ra, const int64_t* __restrict__ ca, const int64_t* __restrict__ rb,
    const int64_t* __restrict__ cb, const int64_t* __restrict__ rc, const int64_t* __restrict__ cc,
    const RowStrides st, int run) {
  using Acc = typename RowMfma<T>::Acc;
  constexpr int RV = 16 / static_cast<int>(sizeof(T));
  constexpr int RB = 16 * RV;                    // rows per block
  constexpr int KP = 4 * KS;
  constexpr int NP = 16 * TN;
  constexpr int ROWB = NP * static_cast<int>(sizeof(T));
  constexpr int SHIFT = 16 * static_cast<int>(sizeof(T));
  constexpr int PADB = ((SHIFT - ROWB % 256 + 256) % 256) / static_cast<int>(sizeof(T));
  __shared__ T Bs[KP][NP + PADB];
  __shared__ int64_t cols_a[KP], cols_c[NP];
  const int64_t q = blockIdx.y;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int e = tid; e < KP * NP; e += 64 * kRowWaves) {
    const int k = e / NP, n = e - (e / NP) * NP;
    T x = T(0);
    if (k < K && n < N) x = B[rb ? rb[q * K + k] + cb[q * N + n] : q * st.bq + k * st.br + n * st.bc];
    Bs[k][n] = x;
  }
  // (past K: the last column again, multiplied by B's zero rows only after a select)
  for (int k = tid; k < KP; k += 64 * kRowWaves) {
    const int kc = min(k, K - 1);
    cols_a[k] = ca ? ca[q * K + kc] : kc * st.ac;
  }
  for (int n = tid; n < N; n += 64 * kRowWaves) cols_c[n] = cc ? cc[q * N + n] : n * st.cc;
  __syncthreads();
  const int kq = lane >> 4;
  const int p = RV * (lane & 15);                // this lane's rows p .. p + RV - 1 of a block
  constexpr int KO = sizeof(T) == 4 ? 4 : 1;
  static_assert(KS % KO == 0, "whole groups of K-steps");
  auto kidx = [&](int s) { return KO > 1 ? 4 * KO * (s / KO) + KO * kq + s % KO : 4 * s + kq; };
  const int per_run = (run + RB - 1) / RB;
  const int64_t blocks = static_cast<int64_t>(M / run) * per_run;
  // Runs of whole 128-byte lines stream past L2 (nontemporal stores: 2 x (48 x 48 x
  // 48^3 2^2) f32 90 -> 70 us).  Elsewhere neighbouring blocks share a line, which
  // such stores would write twice (1716 -> 2037 us on runs of 57^3), and XCD x takes
  // the x-th eighth of the blocks (workgroups go round-robin over the 8 XCDs) so that
  // they meet in one L2 (1763 -> 1716 us; whole lines lose by it, 115 -> 123 us)
  const int xcds = gridDim.x % 8 == 0 && !WHOLE ? 8 : 1, xcd = static_cast<int>(blockIdx.x) % xcds;
  const int64_t end = blocks * (xcd + 1) / xcds;
  const int64_t step = static_cast<int64_t>(gridDim.x / xcds) * kRowWaves;
  // block b: its first row and rows inside its run
  auto rows_of = [&](int64_t b, int& valid) {
    const int j = static_cast<int>(b / per_run), i = static_cast<int>(b - static_cast<int64_t>(j) * per_run);
    valid = min(RB, run - i * RB);
    return j * run + i * RB;
  };
  using AV = RowVec<T, RV>;
  auto load_a = [&](int64_t b, AV (&a)[KS]) {
    int valid;
    const int m = rows_of(b, valid);
    const T* base = A + (ra ? ra[q * M + m] : q * st.aq + m * st.ar) + p;
    if (valid == RB) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        a[s] = *reinterpret_cast<const AV*>(base + cols_a[kidx(s)]);
      }
    } else {
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int t = 0; t < RV; ++t) a[s].v[t] = p + t < valid ? base[cols_a[kidx(s)] + t] : T(0);
    }
    // past K: zeros (B's rows there are zero too)
    if (K < KP) {
#pragma unroll
      for (int s = 0; s < KS; ++s)
        if (kidx(s) >= K)
#pragma unroll
          for (int t = 0; t < RV; ++t) a[s].v[t] = T(0);
    }
  };
  int64_t blk = blocks * xcd / xcds + static_cast<int64_t>(blockIdx.x / xcds) * kRowWaves + wave;
  for (; blk < end; blk += step) {
    AV a[KS];
    load_a(blk, a);
    Acc acc[RV][TN];
#pragma unroll
    for (int t = 0; t < RV; ++t)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[t][j] = Acc{};
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const T b = Bs[kidx(s)][j * 16 + (lane & 15)];
#pragma unroll
        for (int t = 0; t < RV; ++t) acc[t][j] = RowMfma<T>::run(b, a[s].v[t], acc[t][j]);
      }
    int valid;
    const int m = rows_of(blk, valid);
    T* out = C + (rc ? rc[q * M + m] : q * st.cq + m * st.cr) + p;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int col = j * 16 + RowMfma<T>::row(lane, r);
        if (col >= N) continue;
        T* o = out + cols_c[col];
        if (valid == RB) {
          AV x;
#pragma unroll
          for (int t = 0; t < RV; ++t) x.v[t] = acc[t][j][r];
          if constexpr (WHOLE) {
            typedef T NV __attribute__((ext_vector_type(RV), aligned(sizeof(T))));
            __builtin_nontemporal_store(__builtin_bit_cast(NV, x), reinterpret_cast<NV*>(o));
          } else {
            *reinterpret_cast<AV*>(o) = x;
          }
        } else {
#pragma unroll
          for (int t = 0; t < RV; ++t)
            if (p + t < valid) o[t] = acc[t][j][r];
        }
      }
  }
}

template <typename T, int KS, int TN>
hipError_t launch_row_runs(int64_t batch, int M, int N, int K, const T* A, const T* B, T* C, hipStream_t s,
                           const FusedTables* f, const RowStrides& st, int run) {
  static const int resident = [] {            // (both forms: the same registers and LDS)
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_gemm_row_runs<T, KS, TN, false>, 64 * kRowWaves, 0) !=
            hipSuccess ||
        per_cu < 1) {
      (void)hipGetLastError();
      per_cu = 2;
    }
    return per_cu * 256;
  }();
  constexpr int RB = 16 * 16 / static_cast<int>(sizeof(T));
  const int64_t blocks = static_cast<int64_t>(M / run) * ((run + RB - 1) / RB);
  const int64_t want = std::max<int64_t>(1, resident / std::max<int64_t>(batch, 1));
  unsigned gx = static_cast<unsigned>(std::min<int64_t>((blocks + kRowWaves - 1) / kRowWaves, want));
  if (gx > 8) gx = (gx + 7) / 8 * 8;
  const bool whole = static_cast<int64_t>(run) * sizeof(T) % 128 == 0 && (reinterpret_cast<uintptr_t>(C) & 127) == 0;
  auto kern = whole ? k_gemm_row_runs<T, KS, TN, true> : k_gemm_row_runs<T, KS, TN, false>;
  hipLaunchKernelGGL(kern, dim3(gx, static_cast<unsigned>(batch)), dim3(64 * kRowWaves), 0, s, A, B, C, M, N, K, f->ra,
                     f->ca, f->rb, f->cb, f->rc, f->cc, st, run);
  return hipGetLastError();
}

template <typename T, int KS>
hipError_t launch_row_runs_ks(int tn, int64_t batch, int M, int N, int K, const T* A, const T* B, T* C, hipStream_t s,
                              const FusedTables* f, const RowStrides& st, int run) {
  switch (tn) {
    case 1: return launch_row_runs<T, KS, 1>(batch, M, N, K, A, B, C, s, f, st, run);
    case 2: return launch_row_runs<T, KS, 2>(batch, M, N, K, A, B, C, s, f, st, run);
    case 3: return launch_row_runs<T, KS, 3>(batch, M, N, K, A, B, C, s, f, st, run);
    default: return launch_row_runs<T, KS, 4>(batch, M, N, K, A, B, C, s, f, st, run);
  }
}

template <typename T, int KS, int TN, bool TR, int RV, int KV = 1>
hipError_t launch_ks_tn(int64_t batch, int M, int N, int K, const T* A, const T* B, T* C, hipStream_t s,
                        const FusedTables* f, const RowStrides& st) {
  const int64_t* ra = f->ra;
  const int64_t* ca = f->ca;
  const int64_t* rb = f->rb;
  const int64_t* cb = f->cb;
  const int64_t* rc = f->rc;
  const int64_t* cc = f->cc;
  // one wave of resident workgroups over all Q (occupancy x 256 CUs), so that
  // each wave walks several row blocks with B loaded once and the next block's
  // loads in flight
  static const int resident = [] {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_gemm_rows<T, KS, TN, TR, RV, KV>, 64 * kRowWaves, 0) !=
            hipSuccess ||
        per_cu < 1) {
      (void)hipGetLastError();
      per_cu = 2;
    }
    return per_cu * 256;
  }();
  constexpr int rows = RV > 1 ? 16 * RV : 16 * row_groups<T, KS, TN>();
  const int64_t blocks = (M + rows - 1) / rows;
  const int64_t want = std::max<int64_t>(1, resident / std::max<int64_t>(batch, 1));
  const unsigned gx = static_cast<unsigned>(std::min<int64_t>((blocks + kRowWaves - 1) / kRowWaves, want));
  hipLaunchKernelGGL((k_gemm_rows<T, KS, TN, TR, RV, KV>), dim3(gx, static_cast<unsigned>(batch)), dim3(64 * kRowWaves),
                     0, s, A, B, C, M, N, K, ra, ca, rb, cb, rc, cc, st);
  return hipGetLastError();
}

template <typename T, int KS, bool TR>
hipError_t launch_ks(int tn, int64_t batch, int M, int N, int K, const T* A, const T* B, T* C, hipStream_t s,
                     const FusedTables* f, const RowStrides& st) {
  // K-major A whose output-mode runs hold 16-byte chunks (f->vec > 1 then): row
  // vectors, binary32 only (four rows per load; binary64's pairs measured no faster)
  constexpr int VE = static_cast<int>(16 / sizeof(T));
  if constexpr (!TR && sizeof(T) == 4) {
    if (f->at && f->vec > 1 && M % VE == 0) {
      switch (tn) {
        case 1: return launch_ks_tn<T, KS, 1, TR, VE>(batch, M, N, K, A, B, C, s, f, st);
        case 2: return launch_ks_tn<T, KS, 2, TR, VE>(batch, M, N, K, A, B, C, s, f, st);
        case 3: return launch_ks_tn<T, KS, 3, TR, VE>(batch, M, N, K, A, B, C, s, f, st);
        default: return launch_ks_tn<T, KS, 4, TR, VE>(batch, M, N, K, A, B, C, s, f, st);
      }
    }
  }
  // A's K index contiguous in aligned runs of 16 bytes (U_al, or U's trailing
  // contracted block): K vectors, binary32 only
  if constexpr (sizeof(T) == 4 && KS % VE == 0) {
    if ((f->ra ? f->a_krow != 0 : st.ac == 1) && K % VE == 0 &&
        (reinterpret_cast<uintptr_t>(A) & 15) == 0) {
      switch (tn) {
        case 1: return launch_ks_tn<T, KS, 1, TR, 1, VE>(batch, M, N, K, A, B, C, s, f, st);
        case 2: return launch_ks_tn<T, KS, 2, TR, 1, VE>(batch, M, N, K, A, B, C, s, f, st);
        case 3: return launch_ks_tn<T, KS, 3, TR, 1, VE>(batch, M, N, K, A, B, C, s, f, st);
        default: return launch_ks_tn<T, KS, 4, TR, 1, VE>(batch, M, N, K, A, B, C, s, f, st);
      }
    }
  }
  switch (tn) {
    case 1: return launch_ks_tn<T, KS, 1, TR, 1>(batch, M, N, K, A, B, C, s, f, st);
    case 2: return launch_ks_tn<T, KS, 2, TR, 1>(batch, M, N, K, A, B, C, s, f, st);
    case 3: return launch_ks_tn<T, KS, 3, TR, 1>(batch, M, N, K, A, B, C, s, f, st);
    default: return launch_ks_tn<T, KS, 4, TR, 1>(batch, M, N, K, A, B, C, s, f, st);
  }
}

template <typename T, bool TR>
hipError_t launch_tr(int64_t batch, int M, int N, int K, const T* a, const T* b, T* c, hipStream_t s,
                     const FusedTables* f, const RowStrides& st) {
  const int tn = (N + 15) / 16;
  const int ks = (K + 3) / 4;
  if (ks <= 4) return launch_ks<T, 4, TR>(tn, batch, M, N, K, a, b, c, s, f, st);
  if (ks <= 8) return launch_ks<T, 8, TR>(tn, batch, M, N, K, a, b, c, s, f, st);
  if (ks <= 12) return launch_ks<T, 12, TR>(tn, batch, M, N, K, a, b, c, s, f, st);
  return launch_ks<T, 16, TR>(tn, batch, M, N, K, a, b, c, s, f, st);
}

template <typename T>
hipError_t launch_typed_rows(int64_t batch, int M, int N, int K, const void* A, const void* B, void* C,
                             hipStream_t s, const FusedTables* f, const RowStrides& st, int run) {
  const T* a = static_cast<const T*>(A);
  const T* b = static_cast<const T*>(B);
  T* c = static_cast<T*>(C);
  // rows contiguous in A and C, in runs that fill three quarters of their blocks
  constexpr int RB = 16 * 16 / static_cast<int>(sizeof(T));
  if (run > 0 && 4 * static_cast<int64_t>(run) >= 3 * ((static_cast<int64_t>(run) + RB - 1) / RB) * RB) {
    const int tn = (N + 15) / 16, ks = (K + 3) / 4;
    if (ks <= 4) return launch_row_runs_ks<T, 4>(tn, batch, M, N, K, a, b, c, s, f, st, run);
    if (ks <= 8) return launch_row_runs_ks<T, 8>(tn, batch, M, N, K, a, b, c, s, f, st, run);
    if (ks <= 12) return launch_row_runs_ks<T, 12>(tn, batch, M, N, K, a, b, c, s, f, st, run);
    return launch_row_runs_ks<T, 16>(tn, batch, M, N, K, a, b, c, s, f, st, run);
  }
  return f->c_trans ? launch_tr<T, true>(batch, M, N, K, a, b, c, s, f, st)
                    : launch_tr<T, false>(batch, M, N, K, a, b, c, s, f, st);
}

}  // namespace

// C[q] = A[q] B[q] for K <= 64 and N <= 64 (f64 when f64, else f32); f: the
// operands' offset tables (nullptr, or a null table: aligned row-major forms
// A [Q][M][K], B [Q][K][N], C [Q][M][N]) and f->c_trans, the store layout
// (same values either way).  batch <= 65535.
// swap (M and K at most 64, N long): the transposed product C^T = B^T A^T, its rows
// the columns of B and C, with every operand's tables in the other role.
hipError_t launch_gemm_rows(bool f64, int64_t batch, int M, int N, int K, const void* A, const void* B, void* C,
                            hipStream_t s, const FusedTables* f, bool swap) {
  if (K < 1 || K > 64 || (swap ? M : N) < 1 || (swap ? M : N) > 64 || batch < 1 || batch > 65535 ||
      (swap ? N : M) < 1)
    return hipErrorInvalidValue;
  const int64_t MK = static_cast<int64_t>(M) * K, KN = static_cast<int64_t>(K) * N, MN = static_cast<int64_t>(M) * N;
  FusedTables t = f ? *f : FusedTables{};
  if (!f) t.c_trans = 0;
  if (swap) {
    FusedTables x{};
    x.ra = t.cb;
    x.ca = t.rb;
    x.rb = t.ca;
    x.cb = t.ra;
    x.rc = t.cc;
    x.cc = t.rc;
    // W's columns contiguous (always in the aligned form): lanes along them
    x.c_trans = t.rc ? t.c_cols : 1;
    // columns contiguous in both B and C (V_al and W_al: all N)
    const int64_t vr = t.cb ? t.v_col_run : N, wr = t.cc ? t.w_col_run : N;
    const int run = static_cast<int>(vr < wr ? vr : wr);
    const RowStrides st{KN, 1, N, MK, 1, K, MN, 1, N};
    return f64 ? launch_typed_rows<double>(batch, N, M, K, B, A, C, s, &x, st, run)
               : launch_typed_rows<float>(batch, N, M, K, B, A, C, s, &x, st, run);
  }
  const RowStrides st{MK, K, 1, KN, N, 1, MN, N, 1};
  return f64 ? launch_typed_rows<double>(batch, M, N, K, A, B, C, s, &t, st, 0)
             : launch_typed_rows<float>(batch, M, N, K, A, B, C, s, &t, st, 0);
}

}  // namespace symt
