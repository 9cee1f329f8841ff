// Pieces shared by the f64 / f32 sector-product kernels (gemm.hip, gemm_any.hpp):
// the MFMA forms, W's tables and stores of a finished tile, and stream-K's
// pieces with the kernel that sums them.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <type_traits>

#include "gemm_common.hpp"
#include "sk_index.hpp"

namespace symt {

namespace {

template <typename T>
struct Mfma;
// Accumulator layouts (lane l, item r, column l % 16): the f64 16x16x4 form
// holds row l/16 + 4r, the f32 16x16x4 and bf16 16x16x32 forms row 4(l/16) + r.
template <>
struct Mfma<double> {
  using Acc = d4;
  static __device__ __forceinline__ Acc run(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <>
struct Mfma<float> {
  using Acc = f4;
  static __device__ __forceinline__ Acc run(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// W's offset-table entries of this thread's rows and columns of a tile, loaded
// before the tile's K loop (so their latency hides behind it) and used by
// store_tile_tab.  rows4: W's rows come in contiguous, 16-byte aligned runs of
// a multiple of 4 elements; a binary32 lane then holds 4 consecutive rows of one
// column (rows 4(l/16) .. +3) and writes them with one 16-byte store.
template <int TM, int TN>
struct CTab {
  int64_t row[TM][4];
  int64_t col[TN];
};

template <typename T, int BM, int BN, int WM, int WN, int TM, int TN>
__device__ __forceinline__ void load_ctab(CTab<TM, TN>& t, int M, int N, int64_t q, int m0, int n0,
                                          const int64_t* __restrict__ rc, const int64_t* __restrict__ cc) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wm0 = (wave / WN) * (BM / WM);
  const int wn0 = (wave % WN) * (BN / WN);
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = n0 + wn0 + j * 16 + (lane & 15);
    t.col[j] = col < N ? cc[q * N + col] : 0;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = m0 + wm0 + i * 16 + Mfma<T>::row(lane, r);
      t.row[i][r] = row < M ? rc[q * M + row] : 0;
    }
}

// The same entries for the aligned row-major C.
template <typename T, int BM, int BN, int WM, int WN, int TM, int TN>
__device__ __forceinline__ void affine_ctab(CTab<TM, TN>& t, int M, int N, int64_t q, int m0, int n0) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < TN; ++j) t.col[j] = n0 + (wave % WN) * (BN / WN) + j * 16 + (lane & 15);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      t.row[i][r] = (q * M + m0 + (wave / WN) * (BM / WM) + i * 16 + Mfma<T>::row(lane, r)) * N;
}

template <typename T, int BM, int BN, int WM, int WN, int TM, int TN, typename Acc>
__device__ __forceinline__ void store_tile_tab(T* __restrict__ C, int M, int N, int m0, int n0,
                                               const CTab<TM, TN>& t, bool rows4, const Acc (&acc)[TM][TN]) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wm0 = (wave / WN) * (BM / WM);
  const int wn0 = (wave % WN) * (BN / WN);
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = n0 + wn0 + j * 16 + (lane & 15);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (sizeof(T) == 4) {
        const int row0 = m0 + wm0 + i * 16 + Mfma<T>::row(lane, 0);
        if (rows4 && row0 + 3 < M) {
          if (col < N) *reinterpret_cast<f4*>(C + t.row[i][0] + t.col[j]) = acc[i][j];
          continue;
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm0 + i * 16 + Mfma<T>::row(lane, r);
        if (row < M && col < N) C[t.row[i][r] + t.col[j]] = acc[i][j][r];
      }
    }
  }
}

// Piece of a cut tile in accumulator order: element ((wave*TM + i)*TN + j)*4 + r
// of lane l sits at 64 * that + l, so stores and the fixup's loads coalesce.
template <int TM, int TN, typename T, typename Acc>
__device__ __forceinline__ void store_piece(T* __restrict__ piece, const Acc (&acc)[TM][TN]) {
  const int lane = threadIdx.x & 63;
  T* pw = piece + (threadIdx.x >> 6) * (TM * TN * 4 * 64) + lane;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) pw[((i * TN + j) * 4 + r) * 64] = acc[i][j][r];
}

// Sums the pieces of every tile that stream-K cut, in increasing K order (so
// the result does not depend on scheduling), and writes the tile.  Workgroup
// (tile, chunk) handles the chunk-th of `chunks` equal ranges of the tile's
// elements in accumulator order (a tile spread over many teams -- long K, few
// tiles -- is summed by many workgroups); tiles covered whole by one team
// return at once.  Each element's sum starts from zero and adds the pieces in
// team order: the same arithmetic whatever `chunks` is.
// T: the product's type (accumulator rows); TP, TC: the pieces' and C's types.
template <typename T, int BM, int BN, int WM, int WN, bool FC, typename TP = T, typename TC = T>
__global__ __launch_bounds__(64 * WM * WN) void k_sk_fixup(
    const TP* __restrict__ part, TC* __restrict__ C, int M, int N, int nk, int tiles_m, int tiles_n,
    int64_t ntiles, int ts, int nteam, const int64_t* __restrict__ rc, const int64_t* __restrict__ cc) {
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
  constexpr int E = BM * BN;                      // elements of a tile (= of a piece)
  constexpr int PER_WAVE = TM * TN * 4 * 64;
  const int64_t tile = blockIdx.x;
  const int chunks = static_cast<int>(gridDim.y);
  const int64_t grp = tile / ts;
  const int member = static_cast<int>(tile - grp * ts);
  const int64_t total = ntiles / ts * nk;
  const int64_t x0 = grp * nk, x1 = x0 + nk;
  // last team whose share starts at or before x0 (its share is not empty)
  const int64_t t_first = sk_first_team(x0, total, nteam);
  if (sk_bound(t_first + 1, total, nteam) >= x1) return;
  // teams t_first .. t_last hold the tile's pieces (the last one holds iteration
  // x1 - 1); their piece offsets go to LDS once (-1: a team with an empty share)
  constexpr int kList = 1024;
  __shared__ int64_t list[kList];
  const int64_t n_teams = sk_first_team(x1 - 1, total, nteam) - t_first + 1;
  const bool listed = n_teams <= kList;
  if (listed) {
    for (int k = static_cast<int>(threadIdx.x); k < n_teams; k += static_cast<int>(blockDim.x)) {
      const int64_t t = t_first + k;
      const int64_t b0 = sk_bound(t, total, nteam), b1 = sk_bound(t + 1, total, nteam);
      list[k] = b1 > b0 ? sk_piece(static_cast<int>(t), member, ts, grp, b0 / nk) * E : -1;
    }
    __syncthreads();
  }
  const int tn = static_cast<int>(tile % tiles_n);
  const int64_t t2 = tile / tiles_n;
  const int tm = static_cast<int>(t2 % tiles_m);
  const int64_t q = t2 / tiles_m;
  TC* Cq = C + (FC ? 0 : q * static_cast<int64_t>(M) * N);
  const int per = (E + chunks - 1) / chunks;
  const int e0 = static_cast<int>(blockIdx.y) * per;
  const int e1 = min(E, e0 + per);
  // accumulator order: element ((w * TM + i) * TN + j) * 4 + r of lane l at 64 * that + l
  // destination of element e of the tile (accumulator order), -1 past M or N;
  // W's table entries are requested before the pieces are read
  auto dest = [&](int e) -> int64_t {
    const int w = e / PER_WAVE;
    const int rem = e - w * PER_WAVE;
    const int lane = rem & 63;
    const int ijr = rem >> 6;
    const int r = ijr & 3;
    const int ij = ijr >> 2;
    const int i = ij / TN, j = ij - (ij / TN) * TN;
    const int row = tm * BM + (w / WN) * (BM / WM) + i * 16 + Mfma<T>::row(lane, r);
    const int col = tn * BN + (w % WN) * (BN / WN) + j * 16 + (lane & 15);
    if (row >= M || col >= N) return -1;
    const int64_t crow = FC ? rc[q * M + row] : static_cast<int64_t>(row) * N;
    const int64_t ccol = FC ? cc[q * N + col] : col;
    return crow + ccol;
  };
  constexpr int NT = 64 * WM * WN;
  constexpr int U = 4;                            // elements in flight per thread
  for (int e = e0 + static_cast<int>(threadIdx.x); e < e1; e += U * NT) {
    TP acc[U];
    int64_t dst[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[u] = TP(0);
      dst[u] = e + u * NT < e1 ? dest(e + u * NT) : -1;
    }
    if (listed) {
#pragma unroll 4
      for (int k = 0; k < static_cast<int>(n_teams); ++k) {
        const int64_t off = list[k];
        if (off >= 0) {
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (e + u * NT < e1) acc[u] += part[off + e + u * NT];
        }
      }
    } else {
      for (int64_t t = t_first; t < nteam; ++t) {
        const int64_t b0 = sk_bound(t, total, nteam), b1 = sk_bound(t + 1, total, nteam);
        if (b0 >= x1) break;
        if (b1 == b0) continue;
        const int64_t off = sk_piece(static_cast<int>(t), member, ts, grp, b0 / nk) * E;
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (e + u * NT < e1) acc[u] += part[off + e + u * NT];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (dst[u] >= 0) Cq[dst[u]] = static_cast<TC>(acc[u]);
  }
}

// Workgroups of the fixup: a tile spans about nk / (iterations per team) + 1
// teams' pieces, and its sum goes to enough workgroups that each thread makes one
// pass of four elements (their loads in flight together), more when the tile has
// many pieces, down to one element per thread.
inline dim3 sk_fixup_grid(int64_t ntiles, int ts, int64_t nk, int64_t nteam, int64_t tile_elems, int threads) {
  const int64_t per_team = std::max<int64_t>(1, (ntiles / ts) * nk / nteam);
  const int64_t spans = nk / per_team + 1;
  const int64_t max_chunks = std::max<int64_t>(1, tile_elems / threads);
  const int64_t one_pass = std::max<int64_t>(1, max_chunks / 4);
  return dim3(static_cast<unsigned>(ntiles),
              static_cast<unsigned>(std::min<int64_t>(max_chunks, std::max<int64_t>(one_pass, spans))));
}

// Compute units of the current device (cached per device).
int device_cus() {
  static std::atomic<int> cus[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cus[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
    cus[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

}  // namespace
}  // namespace symt
