// Sector product in place for any layout of its operands (Alg. 2's product step,
// f64 / f32, real or complex): the global-to-LDS ring of gemm.hip's tiles with a
// loader that takes every layout of U, V and W, K runs of any length, and any
// element alignment, so that no aligned form is written and no shape falls back
// to register-staged one-element loads.
//
// What bounds it: the matrix pipes once a tile's loads are in flight, as for the
// other global-to-LDS tiles; what it saves is passes over memory (aligned forms
// of K-major or complex operands) and the issue slots of one-element register
// loads.  Its loads differ from those tiles' in three ways:
//  * CH = 4: each lane copies 4 bytes, so a tile row needs no 16-byte alignment
//    and no whole 16-byte chunk (odd block sizes); four times the load
//    instructions of CH = 16, still few beside a K-step's MFMAs (24 loads of a
//    wave against 36 f64 MFMAs of 64 cycles on 96 x 96).
//  * K tails: lanes past the valid depth of a K-step read a zero word instead
//    (both operands, so that nothing of a neighbouring row is multiplied).
//  * every K row of a K-major A at its own table entry, one scalar load per row
//    and step, issued a step ahead (any layout of U's contracted modes).
// Complex operands run on the real representation of C (include/symtensor.h,
// COMPLEX OPERANDS) without expanding V: B's tile holds V's (re, im) pairs once
// and the odd real rows (-im, re) are formed as fragments are read; A is read as
// interleaved reals (its contracted modes last) or K-major as pairs.
//
// Measured (before -> after): the complex bond-64 environment chain 648 -> 247 us
// (its align passes alone took 392); 9 x (500 x 500 x 500) f64 71.7 -> 64.5 us,
// f32 47.3 -> 37.0 us; the Z_8 ladder in f32 (8 x (4608 x 4608 x 288)) 918 -> 844 us
// (96 x 96 with three workgroups per CU against a 64 x 96 register tile); the
// complex ladder over Z_2 x Z_4 with blocks of 18 and 5 in f64 1985 -> 1722 us, over Z_8 with
// 24 and 6 in f32 3491 -> 3138.  4-byte loads run
// at about two thirds of 16-byte ones' rate (3 x (743 x 1113 x 1111) f64: 34.5
// TFLOP/s), so odd real shapes mostly stay on the register tiles.
//
// BF (binary32 operands): the split-bf16 product.  A fragment's eight values are
// split into hi and lo in registers as they are read (24 VALU operations against
// 3 MFMAs per tile of 16 x 16), so no operand goes to bf16 planes first; two
// binary32 accumulators (hi hi, and the cross terms) as the other tiles of that
// product, pieces of cut tiles in binary64.  It is bound by those splits and the
// eight LDS reads of each B fragment (0.2 to 0.3 of a third of the bf16 peak), so
// large products with whole 32-deep K-steps stay on planes, whose tiles reach 0.9;
// what it saves is the planes' write and reads (12 bytes per element), three or
// four launches, and the single pass over a long K that those tiles make.
// Before -> after, whole contractions: 5 x (120 x 320 x 90) 41 -> 20 us, 4 x (1156 x
// 1156 x 36) 110 -> 32, 6 x (16 x 186624 x 18) 5233 -> 133, 8 x (3200 x 3200 x 128) 343 ->
// 153 (195 before the wide tiles were timed as they run; those take it now, at 164).
//
// Values and K order are the other tiles': K-steps of 128 bytes, four indices
// per MFMA, tiles cut by stream-K summed in K order by k_sk_fixup.  Where K was cut
// before, binary32 sums of 128 indices go to a second accumulator (kAnyChunk: 16 to 36
// additions a chunk, up to 6% of the time on 96 x 96, whose registers it fills).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "any_index.hpp"
#include "gemm_tiles.hpp"
#include "plan.hpp"
#include "sk_index.hpp"

namespace symt {
namespace {

// Source of the lanes past a K-step's valid depth.
__device__ __attribute__((aligned(16))) const uint32_t kZeroWords[4] = {0, 0, 0, 0};

template <int CH>
__device__ __forceinline__ void lds_dma(const void* g, void* lds) {
  static_assert(CH == 16 || CH == 4, "lane load");
  if constexpr (CH == 16) __builtin_amdgcn_global_load_lds((gptr_t)(g), (lptr_t)(lds), 16, 0, 0);
  else __builtin_amdgcn_global_load_lds((gptr_t)(g), (lptr_t)(lds), 4, 0, 0);
}

// K-steps that a binary32 accumulator sums before it starts over (128 indices), where these
// tiles replace a product that cuts K: its sums hold at least 128 indices each, and one
// accumulator over all of K is further off (CK; rms 6.9e-7 against 2.1e-7 at K = 744 complex).
constexpr int kAnyChunk = 4;

// AM, CB: the tile's layouts (any_index.hpp).  Null tables stand for the aligned
// row-major forms (the three-step path, so that it sums in the same order).
template <typename T, int BM, int BN, int WM, int WN, int CH, int AM, bool CB>
struct AnyTile {
  static constexpr int ES = static_cast<int>(sizeof(T));
  static constexpr int NW = WM * WN, NT = 64 * NW;
  static constexpr int VE = 16 / ES;
  static constexpr int BK = 128 / ES;
  static constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
  static constexpr int A_BYTES = BM * 128;
  static constexpr int A_ROW = AM == 0 ? 128 : AM == 1 ? BM * ES : 2 * BM * ES;   // bytes of an LDS row
  static constexpr int B_ROW = BN * ES;
  static constexpr int B_BYTES = (CB ? BK / 2 : BK) * B_ROW;
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int A_LOADS = (A_BYTES / CH + NT - 1) / NT, B_LOADS = (B_BYTES / CH + NT - 1) / NT;
  static_assert(A_BYTES % (64 * CH) == 0 && B_BYTES % (64 * CH) == 0, "loads must fill whole waves");
  static_assert(TM * WM * 16 == BM && TN * WN * 16 == BN, "tile shape");
  using Acc = typename Mfma<T>::Acc;
};

// A tile's sums: one accumulator per 16 x 16 block, two in the split-bf16 product.
template <typename T, int TM, int TN, bool BF>
struct AnyAcc {
  typename Mfma<T>::Acc v[TM][TN];
};
template <int TM, int TN>
struct AnyAcc<float, TM, TN, true> {
  f4 v[TM][TN], x[TM][TN];
};

// Most LDS rows that one wave load (64 lanes of CH bytes) of a tile with ROW-byte rows touches.
template <int CH, int ROW>
constexpr int any_rows_per_load() {
  // (loads start at multiples of gcd(64 CH, ROW) in a row)
  int g = ROW, b = 64 * CH;
  while (b) {
    const int t = g % b;
    g = b;
    b = t;
  }
  return (ROW - g + 64 * CH - 1) / ROW + 1;
}

template <typename T, int BM, int BN, int WM, int WN, int CH, int AM, bool CB, bool BF, bool CK>
__device__ __forceinline__ void any_tile_accumulate(
    const T* __restrict__ A, const T* __restrict__ B, int M, int N, const AnySteps& st, int64_t q, int m0, int n0,
    int kt0, int kt1, const int64_t* __restrict__ ra, const int64_t* __restrict__ ca,
    const int64_t* __restrict__ rb, const int64_t* __restrict__ cb, int64_t ldb, char* smem,
    AnyAcc<T, BM / WM / 16, BN / WN / 16, BF>& acc) {
  using D = AnyTile<T, BM, BN, WM, WN, CH, AM, CB>;
  constexpr int ES = D::ES, NT = D::NT, NW = D::NW, BK = D::BK, TM = D::TM, TN = D::TN;
  constexpr int A_LOADS = D::A_LOADS, B_LOADS = D::B_LOADS, STAGE = D::STAGE, A_BYTES = D::A_BYTES;
  constexpr int A_ROW = D::A_ROW;
  constexpr int A_NR = any_rows_per_load<CH, A_ROW>();
  const int K = st.K;
  const int KB = CB ? K / 2 : K;                 // rows of B's table
  const char* Ab = reinterpret_cast<const char*>(A);
  const char* Bb = reinterpret_cast<const char*>(B) + (rb ? 0 : q * static_cast<int64_t>(K) * N * ES);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / WN) * (BM / WM);
  const int wn0 = (wave % WN) * (BN / WN);

  // Byte offset of each load's source, fixed across K-steps; the K index (AM = 0)
  // or LDS row of the lane inside the step is recomputed where a tail needs it.
  int64_t a_src[A_LOADS], b_src[B_LOADS];
#pragma unroll
  for (int i = 0; i < A_LOADS; ++i) {
    const AnySlot x = any_a_slot<ES, BM, AM, BF && AM != 0>((i * NT + tid) * CH);
    constexpr int PE = AM == 0 ? 16 : AM == 2 ? 2 * ES : ES;   // bytes of one m in a load
    const int m = min(m0 + x.line, any_last_line<CH, PE>(M));
    a_src[i] = (ra ? ra[q * M + m] : (q * M + m) * static_cast<int64_t>(K)) * ES + (AM == 0 || CH == 4 ? x.sub : 0);
  }
#pragma unroll
  for (int i = 0; i < B_LOADS; ++i) {
    const AnySlot x = any_b_slot<ES, BN, CB, BF>((i * NT + tid) * CH);
    const int n = min(n0 + x.line, any_last_line<CH, ES>(N));
    b_src[i] = ((CB ? x.k / 2 : x.k) * ldb + (cb ? cb[q * N + n] : static_cast<int64_t>(n))) * ES +
               (CH == 4 ? x.sub : 0);
  }
  // Table entries of the next step to issue (wave-uniform scalar loads, one step ahead).
  int k0_next = 0, kv_next = 0;
  int64_t acol_next = 0;
  int64_t arow_next[AM ? A_LOADS : 1][AM ? A_NR : 1];
  int64_t brow_next = 0;
  auto fetch = [&](int kt) {
    any_step(st, kt, BK, k0_next, kv_next);
    if constexpr (AM == 0) {
      acol_next = ca ? ca[q * K + k0_next] : k0_next;
    } else {
#pragma unroll
      for (int i = 0; i < A_LOADS; ++i) {
        const int r0 = (i * NW + wave) * 64 * CH / A_ROW;
#pragma unroll
        for (int j = 0; j < A_NR; ++j)
          arow_next[i][j] = ca[q * K + min(k0_next + (AM == 2 ? 2 : 1) * (r0 + j), K - 1)];
      }
    }
    const int kb = CB ? k0_next / 2 : k0_next;
    brow_next = rb ? rb[q * KB + kb] : kb * ldb;
  };
  // K-major A: the entry of this lane's LDS row among those its wave load touches.
  auto arow_of = [&](int i) -> int64_t {
    if constexpr (AM == 0) {
      return acol_next;
    } else {
      const int at = (i * NW + wave) * 64 * CH % A_ROW + lane * CH;
      int64_t off = arow_next[i][0];
#pragma unroll
      for (int j = 1; j < A_NR; ++j) {
        const int64_t e = arow_next[i][j];
        off = at >= j * A_ROW ? e : off;
      }
      return off;
    }
  };
  auto issue = [&](int kt, int stage) {
    char* base = smem + stage * STAGE + wave * 64 * CH;
    const int kv = kv_next;
    const bool tail = kv < BK;
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i) {
      if (A_BYTES % (CH * NT) != 0 && (i * NW + wave) * 64 * CH >= A_BYTES) break;
      const char* g = Ab + (a_src[i] + arow_of(i) * ES);
      if (tail) {
        const int k = any_a_slot<ES, BM, AM, BF && AM != 0>((i * NT + tid) * CH).k;
        if (k >= kv) g = reinterpret_cast<const char*>(kZeroWords);
      }
      lds_dma<CH>(g, base + i * NT * CH);
    }
#pragma unroll
    for (int i = 0; i < B_LOADS; ++i) {
      if (D::B_BYTES % (CH * NT) != 0 && (i * NW + wave) * 64 * CH >= D::B_BYTES) break;
      const char* g = Bb + (b_src[i] + brow_next * ES);
      if (tail) {
        const int k = any_b_slot<ES, BN, CB, BF>((i * NT + tid) * CH).k;
        if (k >= kv) g = reinterpret_cast<const char*>(kZeroWords);
      }
      lds_dma<CH>(g, base + A_BYTES + i * NT * CH);
    }
    if (kt + 1 < kt1) fetch(kt + 1);
  };

  const int nk = kt1 - kt0;
  // CK: the sum of every kAnyChunk K-steps is added to `sum` and starts over
  static_assert(!CK || (std::is_same<T, float>::value && !BF), "binary32 sums");
  typename D::Acc sum[CK ? TM : 1][CK ? TN : 1];
  if constexpr (CK) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) sum[i][j] = typename D::Acc{};
  }
  if (nk > 0) {
    fetch(kt0);
    issue(kt0, 0);
  }
  for (int it = 0; it < nk; ++it) {
    // this wave's loads of step it have landed; past the barrier every wave's have, and
    // every wave is done with the other stage
    wait_vmcnt<0>();
    asm volatile("s_barrier" ::: "memory");
    if (it + 1 < nk) issue(kt0 + it + 1, (it + 1) % 2);
    const char* As = smem + (it % 2) * STAGE;
    const char* Bs = As + A_BYTES;
    if constexpr (BF) {
      const int g = lane >> 4;
      bf8 ah[TM], al[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int m = wm0 + i * 16 + (lane & 15);
        fv4 x[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if constexpr (AM == 0) {
            x[h] = *reinterpret_cast<const fv4*>(As + any_a_off<ES, BM, AM>(m, any_k_bf16(g, 4 * h)));
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              x[h][e] = *reinterpret_cast<const T*>(As + any_a_off<ES, BM, AM, true>(m, any_k_bf16(g, 4 * h + e)));
          }
        }
        split8(x[0], x[1], ah[i], al[i]);
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int n = wn0 + j * 16 + (lane & 15);
        fv4 x[2];
#pragma unroll
        for (int e = 0; e < 8; ++e)
          x[e >> 2][e & 3] = *reinterpret_cast<const T*>(Bs + any_b_off<ES, BN, CB, true>(any_k_bf16(g, e), n));
        bf8 bh, bl;
        split8(x[0], x[1], bh, bl);
        // (the two updates of each cross accumulator are TM products apart)
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          acc.v[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bh, acc.v[i][j], 0, 0, 0);
          acc.x[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bl, acc.x[i][j], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
          acc.x[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[i], bh, acc.x[i][j], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int kk = 0; kk < BK; kk += 4) {
        const int k = kk + (lane >> 4);
        T a[TM], b[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          a[i] = *reinterpret_cast<const T*>(As + any_a_off<ES, BM, AM>(wm0 + i * 16 + (lane & 15), k));
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int n = wn0 + j * 16 + (lane & 15);
          const T x = *reinterpret_cast<const T*>(Bs + any_b_off<ES, BN, CB>(k, n));
          // CB: real row 2 kc + 1 is (-im, re), the other member of the pair, im negated
          b[j] = CB && (k & 1) && !(n & 1) ? -x : x;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc.v[i][j] = Mfma<T>::run(a[i], b[j], acc.v[i][j]);
      }
      if constexpr (CK)
        if (it % kAnyChunk == kAnyChunk - 1) {
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              sum[i][j] += acc.v[i][j];
              acc.v[i][j] = typename D::Acc{};
            }
        }
    }
  }
  if constexpr (CK) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc.v[i][j] += sum[i][j];
  }
}

// Waves per SIMD that the register allocator leaves room for: three where the LDS
// ring admits three workgroups per CU; two with 4-byte loads, whose 24 load
// sources take 48 registers (96 x 96 spilled 73 of them at three).
template <int BM, int BN, int CH, bool BF = false>
constexpr int kAnyWavesPerSimd = BM * BN <= 64 * 64 || (CH == 16 && !BF) ? 3 : 2;

// Split-bf16 sums to W (binary64 sums of the two accumulators, rounded to TC) and to a piece.
template <typename TC, int BM, int BN, int WM, int WN, int TM, int TN>
__device__ __forceinline__ void store_any_bf16(TC* __restrict__ C, int M, int N, int m0, int n0,
                                               const CTab<TM, TN>& t, bool rows4,
                                               const AnyAcc<float, TM, TN, true>& acc) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = n0 + (wave % WN) * (BN / WN) + j * 16 + (lane & 15);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row0 = m0 + (wave / WN) * (BM / WM) + i * 16 + Mfma<float>::row(lane, 0);
      TC v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        v[r] = static_cast<TC>(static_cast<double>(acc.v[i][j][r]) + static_cast<double>(acc.x[i][j][r]));
      if constexpr (sizeof(TC) == 4) {
        if (rows4 && row0 + 3 < M) {
          if (col < N) *reinterpret_cast<f4*>(C + t.row[i][0] + t.col[j]) = f4{v[0], v[1], v[2], v[3]};
          continue;
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (row0 + r < M && col < N) C[t.row[i][r] + t.col[j]] = v[r];
    }
  }
}
template <int TM, int TN>
__device__ __forceinline__ void store_any_piece(double* __restrict__ piece, const AnyAcc<float, TM, TN, true>& acc) {
  const int lane = threadIdx.x & 63;
  double* pw = piece + (threadIdx.x >> 6) * (TM * TN * 4 * 64) + lane;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        pw[((i * TN + j) * 4 + r) * 64] = static_cast<double>(acc.v[i][j][r]) + static_cast<double>(acc.x[i][j][r]);
}

// One workgroup per tile (ts = 0, XCD-aware order), or stream-K (ts > 0:
// persistent workgroups, pieces of cut tiles to `part` for k_sk_fixup).
template <typename T, int BM, int BN, int WM, int WN, int CH, int AM, bool CB, bool BF = false,
          typename TC = T, bool CK = false>
__global__ __launch_bounds__(64 * WM * WN, (kAnyWavesPerSimd<BM, BN, CH, BF>)) void k_gemm_any(
    const T* __restrict__ A, const T* __restrict__ B, TC* __restrict__ C, int M, int N, AnySteps st, int tiles_m,
    int tiles_n, int64_t ntiles, const int64_t* __restrict__ ra, const int64_t* __restrict__ ca,
    const int64_t* __restrict__ rc, const int64_t* __restrict__ cc, const int64_t* __restrict__ rb,
    const int64_t* __restrict__ cb, int64_t ldb,
    typename std::conditional<BF, double, T>::type* __restrict__ part, int ts, int c_rows4) {
  using D = AnyTile<T, BM, BN, WM, WN, CH, AM, CB>;
  constexpr int TM = D::TM, TN = D::TN;
  __shared__ __attribute__((aligned(1024))) char smem[2 * D::STAGE];
  AnyAcc<T, TM, TN, BF> acc;
  SkSlot sl{0, 0, 1};
  int64_t it = 0, end = st.nk, first = 0, tile = 0;
  if (ts > 0) {
    sl = sk_slot(static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x), ts);
    const int64_t total = ntiles / ts * st.nk;
    it = sk_bound(sl.team, total, sl.nteam);
    end = sk_bound(sl.team + 1, total, sl.nteam);
    first = it / st.nk;
  } else {
    tile = xcd_remap(blockIdx.x, ntiles);
  }
  while (it < end) {
    int64_t q, grp = 0;
    int tm, tn, kt0 = 0, kt1 = st.nk;
    if (ts > 0) {
      grp = it / st.nk;
      kt0 = static_cast<int>(it - grp * st.nk);
      kt1 = static_cast<int>(min(static_cast<int64_t>(st.nk), kt0 + (end - it)));
      tile = grp * ts + sl.member;
      tn = static_cast<int>(tile % tiles_n);
      const int64_t t2 = tile / tiles_n;
      tm = static_cast<int>(t2 % tiles_m);
      q = t2 / tiles_m;
      __syncthreads();      // the previous piece's LDS reads are done before new loads land
    } else {
      tile_coords(tile, tiles_m, tiles_n, q, tm, tn);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        acc.v[i][j] = typename D::Acc{};
        if constexpr (BF) acc.x[i][j] = typename D::Acc{};
      }
    any_tile_accumulate<T, BM, BN, WM, WN, CH, AM, CB, BF, CK>(A, B, M, N, st, q, tm * BM, tn * BN, kt0, kt1, ra,
                                                                  ca, rb, cb, ldb, smem, acc);
    if (kt0 == 0 && kt1 == st.nk) {
      // W's table entries all requested before the first store
      CTab<TM, TN> ct;
      if (rc) load_ctab<T, BM, BN, WM, WN, TM, TN>(ct, M, N, q, tm * BM, tn * BN, rc, cc);
      else affine_ctab<T, BM, BN, WM, WN, TM, TN>(ct, M, N, q, tm * BM, tn * BN);
      if constexpr (BF)
        store_any_bf16<TC, BM, BN, WM, WN, TM, TN>(C, M, N, tm * BM, tn * BN, ct, c_rows4 != 0, acc);
      else
        store_tile_tab<T, BM, BN, WM, WN, TM, TN>(C, M, N, tm * BM, tn * BN, ct, c_rows4 != 0, acc.v);
    } else {
      auto* piece = part + sk_piece(sl.team, sl.member, ts, grp, first) * (BM * BN);
      if constexpr (BF) store_any_piece<TM, TN>(piece, acc);
      else store_piece<TM, TN>(piece, acc.v);
    }
    it += kt1 - kt0;
  }
}

template <typename T, int BM, int BN, int WM, int WN, int CH, int AM, bool CB, bool BF = false,
          typename TC = T, bool CK = false>
hipError_t launch_any_kernel(int64_t batch, int M, int N, const AnySteps& st, const void* A, const void* B, void* C,
                             hipStream_t s, const FusedTables* f, void* part, size_t part_bytes, bool sk) {
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  const int64_t ntiles = batch * tiles_m * tiles_n;
  const dim3 block(64 * WM * WN);
  const T* a = static_cast<const T*>(A);
  const T* b = static_cast<const T*>(B);
  using TP = typename std::conditional<BF, double, T>::type;
  TC* c = static_cast<TC*>(C);
  TP* pt = static_cast<TP*>(part);
  const int rows4 = f->c_rows4 && (reinterpret_cast<uintptr_t>(c) & 15) == 0 ? 1 : 0;
  auto kern = k_gemm_any<T, BM, BN, WM, WN, CH, AM, CB, BF, TC, CK>;
  int P = 0, ts = 0;
  if (sk && part) {
    // (as many per CU as every layout of this tile and load width admits: the in-place
    // product and the three steps share K out alike)
    constexpr int wgs = kAnyWavesPerSimd<BM, BN, CH, BF>;
    const SkLaunch sl = sk_launch(ntiles, tiles_n, st.nk, std::min<int64_t>(kSkSlots, static_cast<int64_t>(device_cus()) * wgs),
                                  static_cast<int64_t>(part_bytes / sizeof(TP)), static_cast<int64_t>(BM) * BN,
                                  kSkMinIters);
    P = sl.P;
    if (P > 0) ts = sl.ts;
  }
  hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(P > 0 ? P : ntiles)), block, 0, s, a, b, c, M, N, st, tiles_m,
                     tiles_n, ntiles, f->ra, f->ca, f->rc, f->cc, f->rb, f->cb, f->rb ? f->ldb : N, pt, ts, rows4);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || P == 0) return e;
  const dim3 fgrid = sk_fixup_grid(ntiles, ts, st.nk, P / ts, static_cast<int64_t>(BM) * BN, 64 * WM * WN);
  if (f->rc)
    hipLaunchKernelGGL((k_sk_fixup<T, BM, BN, WM, WN, true, TP, TC>), fgrid, block, 0, s, pt, c, M, N, st.nk, tiles_m, tiles_n,
                       ntiles, ts, P / ts, f->rc, f->cc);
  else
    hipLaunchKernelGGL((k_sk_fixup<T, BM, BN, WM, WN, false, TP, TC>), fgrid, block, 0, s, pt, c, M, N, st.nk, tiles_m,
                       tiles_n, ntiles, ts, P / ts, f->rc, f->cc);
  return hipGetLastError();
}

// Tiles in the order of the planner's table (the 96 x 96 one takes 16-byte loads
// only: with 4-byte loads its sources and accumulators exceed two waves' registers).
template <typename T, int CH, int AM, bool CB, bool CK>
hipError_t launch_any_tile(const AnyLaunch& l, int64_t batch, int M, int N, const AnySteps& st, const void* A,
                           const void* B, void* C, hipStream_t s, const FusedTables* f, void* part, size_t part_bytes) {
  if constexpr (CH == 16)
    if (l.tile == 0)
      return launch_any_kernel<T, 96, 96, 2, 2, CH, AM, CB, false, T, CK>(batch, M, N, st, A, B, C, s, f, part,
                                                                           part_bytes, l.sk);
  if (l.tile <= 1)
    return launch_any_kernel<T, 128, 64, 2, 2, CH, AM, CB, false, T, CK>(batch, M, N, st, A, B, C, s, f, part,
                                                                          part_bytes, l.sk);
  return launch_any_kernel<T, 64, 64, 2, 2, CH, AM, CB, false, T, CK>(batch, M, N, st, A, B, C, s, f, part,
                                                                       part_bytes, l.sk);
}

template <typename T, int CH, bool CK>
hipError_t launch_any_typed(const AnyLaunch& l, int64_t batch, int M, int N, const AnySteps& st, const void* A,
                            const void* B, void* C, hipStream_t s, const FusedTables* f, void* part,
                            size_t part_bytes) {
  if (l.cb)
    return l.am == 0 ? launch_any_tile<T, CH, 0, true, CK>(l, batch, M, N, st, A, B, C, s, f, part, part_bytes)
                     : launch_any_tile<T, CH, 2, true, CK>(l, batch, M, N, st, A, B, C, s, f, part, part_bytes);
  return l.am == 0 ? launch_any_tile<T, CH, 0, false, CK>(l, batch, M, N, st, A, B, C, s, f, part, part_bytes)
                   : launch_any_tile<T, CH, 1, false, CK>(l, batch, M, N, st, A, B, C, s, f, part, part_bytes);
}

}  // namespace
}  // namespace symt
