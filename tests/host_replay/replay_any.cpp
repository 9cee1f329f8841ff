// Host replay of the in-place product for any layout: plans random contractions
// with its tiles forced, rebuilds each tile's LDS image load by load with the
// kernel's own index functions (csrc/any_index.hpp), and checks that every load
// stays inside its operand and aligned, and that every MFMA operand read finds
// the element that the plan's offset tables name (zero past a K-step's depth).
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <numeric>
#include <string>
#include <vector>

#include "any_index.hpp"
#include "plan.hpp"
#include "xform_index.hpp"

using namespace symt;

static int64_t g_checks = 0, g_fail = 0, g_plans = 0, g_tails = 0, g_am[3] = {}, g_cb = 0, g_odd = 0, g_bf = 0, g_direct = 0, g_clear = 0;
static std::string g_case;
#define CHECK(c, what, x, y)                                                                            \
  do {                                                                                                  \
    ++g_checks;                                                                                         \
    if (!(c)) {                                                                                         \
      if (++g_fail <= 20)                                                                               \
        std::printf("FAIL %s: %s (%lld, %lld)\n", g_case.c_str(), what, static_cast<long long>(x),      \
                    static_cast<long long>(y));                                                         \
    }                                                                                                   \
  } while (0)

struct Rng {
  uint64_t s;
  uint32_t next() {
    s = s * 6364136223846793005ull + 1442695040888963407ull;
    return static_cast<uint32_t>(s >> 33);
  }
  int below(int n) { return static_cast<int>(next() % static_cast<uint32_t>(n)); }
};

static std::vector<int64_t> table(const OffsetParams& o, int G) {
  std::vector<int64_t> t(static_cast<size_t>(G) * o.count);
  for (int q = 0; q < G; ++q)
    for (int64_t i = 0; i < o.count; ++i) t[q * o.count + i] = table_entry(o, q, i);
  return t;
}

// One tile shape on one plan: the first and last tile of every slice.
template <int ES, int BM, int BN, int CH, int AM, bool CB, bool BF = false>
void replay_tile(const Plan& p, const std::vector<int64_t>& ra, const std::vector<int64_t>& ca,
                 const std::vector<int64_t>& rb, const std::vector<int64_t>& cb) {
  constexpr int BK = 128 / ES;
  constexpr int A_BYTES = BM * 128, B_BYTES = (CB ? BK / 2 : BK) * BN * ES;
  const int M = static_cast<int>(p.M), N = static_cast<int>(p.gn), K = static_cast<int>(p.gk);
  const AnySteps st = any_steps(K, p.any.krun, BK);
  const int KB = CB ? K / 2 : K;
  const int64_t a_bytes = p.U.elems * (p.cplx ? 2 : 1) * ES;
  const int64_t b_bytes = (p.any.b ? p.V.elems * (p.cplx ? 2 : 1) : static_cast<int64_t>(p.g.size) * K * N) * ES;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  const int64_t ldb = p.any.b ? p.any.ldb : N;
  std::vector<int64_t> la(A_BYTES / 4), lb(B_BYTES / 4);
  for (int64_t q = 0; q < p.g.size; ++q)
    for (int e = 0; e < 2; ++e) {
      const int m0 = (e ? tiles_m - 1 : 0) * BM, n0 = (e ? tiles_n - 1 : 0) * BN;
      int covered = 0;
      for (int kt = 0; kt < st.nk; ++kt) {
        int k0, kv;
        any_step(st, kt, BK, k0, kv);
        CHECK(k0 == covered && kv > 0 && k0 + kv <= K, "K-steps not in order", k0, kv);
        covered = k0 + kv;
        g_tails += kv < BK;
        constexpr int PE = AM == 0 ? 16 : AM == 2 ? 2 * ES : ES;
        for (int at = 0; at < A_BYTES; at += CH) {
          const AnySlot x = any_a_slot<ES, BM, AM, BF && AM != 0>(at);
          const int m = std::min(m0 + x.line, any_last_line<CH, PE>(M));
          const int64_t col = AM == 0 ? ca[q * K + k0] : ca[q * K + std::min(k0 + x.k, K - 1)];
          int64_t src = (ra[q * M + m] + col) * ES + (AM == 0 || CH == 4 ? x.sub : 0);
          if (x.k >= kv) src = -1;
          else {
            CHECK(src >= 0 && src + CH <= a_bytes, "A load out of U", src, a_bytes);
            CHECK(CH == 4 || src % 16 == 0, "A load not aligned", src, CH);
          }
          for (int d = 0; d < CH / 4; ++d) la[at / 4 + d] = src < 0 ? -1 : src / 4 + d;
        }
        for (int at = 0; at < B_BYTES; at += CH) {
          const AnySlot x = any_b_slot<ES, BN, CB, BF>(at);
          const int n = std::min(n0 + x.line, any_last_line<CH, ES>(N));
          const int kb = CB ? k0 / 2 : k0;
          const int64_t base = p.any.b ? rb[q * KB + kb] : q * static_cast<int64_t>(K) * N + kb * ldb;
          int64_t src = (base + (CB ? x.k / 2 : x.k) * ldb + (p.any.b ? cb[q * N + n] : n)) * ES +
                        (CH == 4 ? x.sub : 0);
          if (x.k >= kv) src = -1;
          else {
            CHECK(src >= 0 && src + CH <= b_bytes, "B load out of V", src, b_bytes);
            CHECK(CH == 4 || src % 16 == 0, "B load not aligned", src, CH);
          }
          for (int d = 0; d < CH / 4; ++d) lb[at / 4 + d] = src < 0 ? -1 : src / 4 + d;
        }
        for (int m = 0; m < BM && m0 + m < M; ++m)
          for (int k = 0; k < BK; ++k) {
            const int off = any_a_off<ES, BM, AM, BF && AM != 0>(m, k);
            CHECK(off >= 0 && off + ES <= A_BYTES && off % ES == 0, "A operand read outside its tile", off, m);
            for (int d = 0; d < ES / 4; ++d) {
              const int64_t want = k < kv ? (ra[q * M + m0 + m] + ca[q * K + k0 + k]) * (ES / 4) + d : -1;
              CHECK(la[off / 4 + d] == want, "A operand is another element", la[off / 4 + d], want);
            }
          }
        for (int n = 0; n < BN && n0 + n < N; ++n)
          for (int k = 0; k < BK; ++k) {
            const int off = any_b_off<ES, BN, CB, BF>(k, n);
            CHECK(off >= 0 && off + ES <= B_BYTES && off % ES == 0, "B operand read outside its tile", off, n);
            int64_t el = -1;
            if (k < kv) {
              if (CB) el = rb[q * KB + (k0 + k) / 2] + cb[q * N + ((n0 + n) ^ (k & 1))];
              else el = p.any.b ? rb[q * K + k0 + k] + cb[q * N + n0 + n] : (q * K + k0 + k) * static_cast<int64_t>(N) + n0 + n;
            }
            for (int d = 0; d < ES / 4; ++d) {
              const int64_t want = el < 0 ? -1 : el * (ES / 4) + d;
              CHECK(lb[off / 4 + d] == want, "B operand is another element", lb[off / 4 + d], want);
            }
          }
      }
      CHECK(covered == K, "K-steps do not cover K", covered, K);
    }
}

template <int ES, int CH, int AM, bool CB>
void replay_tiles(const Plan& p, const std::vector<int64_t>& ra, const std::vector<int64_t>& ca,
                  const std::vector<int64_t>& rb, const std::vector<int64_t>& cb) {
  if (p.any.tile == 0 && CH == 16) replay_tile<ES, 96, 96, CH, AM, CB>(p, ra, ca, rb, cb);
  else if (p.any.tile <= 1) replay_tile<ES, 128, 64, CH, AM, CB>(p, ra, ca, rb, cb);
  else replay_tile<ES, 64, 64, CH, AM, CB>(p, ra, ca, rb, cb);
}
template <int ES, int CH>
void replay_layouts(const Plan& p, const std::vector<int64_t>& ra, const std::vector<int64_t>& ca,
                    const std::vector<int64_t>& rb, const std::vector<int64_t>& cb) {
  if (p.any.cb) {
    if (p.any.am == 0) replay_tiles<ES, CH, 0, true>(p, ra, ca, rb, cb);
    else replay_tiles<ES, CH, 2, true>(p, ra, ca, rb, cb);
  } else {
    if (p.any.am == 0) replay_tiles<ES, CH, 0, false>(p, ra, ca, rb, cb);
    else replay_tiles<ES, CH, 1, false>(p, ra, ca, rb, cb);
  }
}

// The split-bf16 tiles; their fragments' K indices cover a step once, and a
// row-major A's come as 16-byte chunks.
template <int CH, int AM>
void replay_bf16(const Plan& p, const std::vector<int64_t>& ra, const std::vector<int64_t>& ca,
                 const std::vector<int64_t>& rb, const std::vector<int64_t>& cb) {
  if (p.any.tile == 0) replay_tile<4, 128, 128, CH, AM, false, true>(p, ra, ca, rb, cb);
  else if (p.any.tile == 1) replay_tile<4, 128, 64, CH, AM, false, true>(p, ra, ca, rb, cb);
  else replay_tile<4, 64, 64, CH, AM, false, true>(p, ra, ca, rb, cb);
  unsigned seen = 0;
  for (int g = 0; g < 4; ++g)
    for (int j = 0; j < 8; ++j) {
      const int k = any_k_bf16(g, j);
      seen |= 1u << k;
      for (int m = 0; m < 16; ++m)
        CHECK((any_a_off<4, 64, 0>)(m, k) - (any_a_off<4, 64, 0>)(m, any_k_bf16(g, j & 4)) == 4 * (j & 3) &&
                  (any_a_off<4, 64, 0>)(m, any_k_bf16(g, j & 4)) % 16 == 0, "A fragment is not whole chunks", m, k);
    }
  CHECK(seen == ~0u, "fragments do not cover the step", seen, 0);
}

static void replay_plan(const Plan& p) {
  ++g_plans;
  ++g_am[p.any.am];
  g_cb += p.any.cb;
  g_odd += !p.any.ch16;
  CHECK(!(p.any.am == 2 && !p.any.cb) && !(p.any.am == 1 && p.any.cb), "layouts without a kernel", p.any.am, p.any.cb);
  const int G = p.g.size;
  const auto ra = table(make_offsets(p, 0, true), G), ca = table(make_offsets(p, 0, false), G);
  std::vector<int64_t> rb, cb;
  if (p.any.b) {
    rb = table(make_offsets(p, 1, true), G);
    cb = table(make_offsets(p, 1, false), G);
    CHECK(rb.size() <= static_cast<size_t>(G) * p.gk && cb.size() == static_cast<size_t>(G) * p.gn, "V's tables",
          rb.size(), cb.size());
  }
  CHECK(p.bytes_partial >= p.any.partial_bytes, "no room for the pieces", p.bytes_partial, p.any.partial_bytes);
  if (p.compute == SYMT_COMPUTE_F64) {
    if (p.any.ch16) replay_layouts<8, 16>(p, ra, ca, rb, cb);
    replay_layouts<8, 4>(p, ra, ca, rb, cb);
  } else if (p.compute == SYMT_COMPUTE_BF16X3) {
    ++g_bf;
    if (p.any.am == 0) {
      if (p.any.ch16) replay_bf16<16, 0>(p, ra, ca, rb, cb);
      replay_bf16<4, 0>(p, ra, ca, rb, cb);
    } else {
      if (p.any.ch16) replay_bf16<16, 1>(p, ra, ca, rb, cb);
      replay_bf16<4, 1>(p, ra, ca, rb, cb);
    }
  } else {
    if (p.any.ch16) replay_layouts<4, 16>(p, ra, ca, rb, cb);
    replay_layouts<4, 4>(p, ra, ca, rb, cb);
  }
}

// The workspace holds what a fused launch lays out in it, in order: U_al (where U
// is aligned), V_al, the offset tables (V's too where the product reads V in
// place) and the pieces; a plan that the product does not take keeps none of its
// layout.
static void check_workspace(const Plan& p) {
  CHECK(p.any.tile >= 0 || (!p.any.b && !p.any.cb && p.any.partial_bytes == 0), "layout of a product not taken",
        p.any.tile, p.any.b);
  if (!(p.fused || p.fused_ua || p.any_direct)) return;
  const size_t G = static_cast<size_t>(p.slices ? p.nq : p.g.size);
  const bool any = p.any.tile >= 0;
  size_t need = p.fused_ua && !any ? round_up(p.ws_u_al, 256) : 0;
  need += (any && p.any.b ? 0 : round_up(p.ws_v_al, 256)) + 2 * round_up(8 * G * p.M, 256) + round_up(8 * G * p.gk, 256) +
          round_up(8 * G * p.gn, 256);
  if (p.fused_b || (any && p.any.b)) need += round_up(8 * G * p.gk, 256) + round_up(8 * G * p.gn, 256);
  need += round_up(p.bytes_partial, 256) + round_up(p.bytes_charges, 256);
  CHECK(need <= p.workspace, "launch layout past the workspace", need, p.workspace);
}

// A subgroup contraction planned over its live slices: every block that the three
// steps' transforms move lies where the offset tables put it, and W is cleared
// exactly where some of its blocks are not reached.
static void check_direct(const Plan& p) {
  const Plan& d = *p.direct;
  ++g_direct;
  g_clear += d.clear_w;
  CHECK(!p.fused && !p.fused_ua && p.any.tile < 0 && d.slices && d.nq == p.nq, "direct plan", p.fused, d.nq);
  CHECK(p.workspace >= d.workspace && p.workspace >= p.workspace_steps, "workspace", p.workspace, d.workspace);
  for (int op = 0; op < 3; ++op) {
    const OffsetParams R = make_offsets(d, op, true), C = make_offsets(d, op, false);
    const XformParams x = make_xform(d, op, true, 8, 8, false, true);
    std::vector<int64_t> seen;
    for (int64_t blk = 0; blk < x.nblocks; ++blk) {
      int64_t sb = -1, ab = -1;
      const bool ok = block_bases(x, blk, sb, ab);
      CHECK(ok, "a live block without a solution", op, blk);
      const int64_t cs = blk % x.gpow_col, rs = blk / x.gpow_col % x.gpow_row;
      const int q = static_cast<int>(blk / x.gpow_col / x.gpow_row);
      const int64_t at = table_entry(R, q, rs * R.n_inner) + table_entry(C, q, cs * C.n_inner * (d.cplx ? 2 : 1));
      CHECK(at == sb, "table entry of a block", at, sb);
      seen.push_back(sb);
    }
    std::sort(seen.begin(), seen.end());
    CHECK(std::adjacent_find(seen.begin(), seen.end()) == seen.end(), "blocks not distinct", op, x.nblocks);
    if (op == 2)
      CHECK((static_cast<int64_t>(seen.size()) * x.blk_elems == d.W.elems * (d.cplx ? 2 : 1)) == !d.clear_w, "blocks not reached",
            seen.size(), d.clear_w);
  }
}

int main(int argc, char** argv) {
  const int n = argc > 1 ? std::atoi(argv[1]) : 200;
  Rng rng{20070805};
  for (int c = 0; c < n; ++c) {
    const int s = 1 + rng.below(2), t = 1 + rng.below(2), v = 1 + rng.below(2);
    const std::string L = "abcdefgh", I = L.substr(0, s), K = L.substr(s, v), J = L.substr(s + v, t);
    std::string tu = rng.below(2) ? I + K : K + I, tv = rng.below(3) ? K + J : J + K, tw = I + J;
    if (rng.below(3) == 0) std::swap(tu[0], tu[rng.below(static_cast<int>(tu.size()))]);
    if (rng.below(3) == 0) std::swap(tw[0], tw[rng.below(static_cast<int>(tw.size()))]);
    symt_group g{};
    g.nfactors = 1 + rng.below(2);
    g.order[0] = 1 + rng.below(4);
    g.order[1] = 2;
    std::vector<int64_t> dim(8);
    for (auto& d : dim) {
      const int r = rng.below(4);
      d = r == 0 ? 1 + rng.below(40) : r == 1 ? 2 * (1 + rng.below(12)) : r == 2 ? 16 : 1 + rng.below(9);
    }
    const bool cplx = rng.below(3) == 0;
    const int compute = rng.below(cplx ? 2 : 3);   // (F64, F32, split-bf16 on binary32)
    const int dt = cplx ? (compute ? SYMT_C64 : SYMT_C128) : (compute ? SYMT_F32 : SYMT_F64);
    auto desc = [&](const std::string& term, std::string& sg, std::vector<int64_t>& dm, bool second) {
      for (char m : term) {
        dm.push_back(dim[m - 'a']);
        const bool neg = (m - 'a') % 2 == 1;
        sg.push_back((second && K.find(m) != std::string::npos ? !neg : neg) ? '-' : '+');
      }
      symt_tensor x{};
      x.nmodes = static_cast<int32_t>(term.size());
      x.signs = sg.c_str();
      x.dims = dm.data();
      x.dtype = dt;
      return x;
    };
    std::string su, sv;
    std::vector<int64_t> du, dv;
    const symt_tensor u = desc(tu, su, du, false), vv = desc(tv, sv, dv, true);
    const std::string sub = tu + "," + tv + "->" + tw;
    for (const char* tile : {"", "a96x96s2", "a128x128s2", "a128x64s2", "a64x64s2"}) {
      if (*tile) setenv("SYMT_GEMM_TILE", tile, 1);
      else unsetenv("SYMT_GEMM_TILE");
      Plan p;
      std::string err;
      // (without a given W the planner takes binary64: bind one of the compute type)
      if (make_plan(sub.c_str(), &g, &u, &vv, nullptr, compute, &p, &err) != SYMT_OK) continue;
      std::string sw;
      std::vector<int64_t> dw;
      for (size_t m = 0; m < tw.size(); ++m) {
        sw.push_back(p.w_sign[m] > 0 ? '+' : '-');
        dw.push_back(dim[tw[m] - 'a']);
      }
      symt_tensor w{};
      w.nmodes = static_cast<int32_t>(tw.size());
      w.signs = sw.c_str();
      w.charge = p.w_charge;
      w.dims = dw.data();
      w.dtype = dt;
      Plan pw;
      if (make_plan(sub.c_str(), &g, &u, &vv, &w, compute, &pw, &err) != SYMT_OK) continue;
      g_case = sub + " " + tile;
      check_workspace(pw);
      if (pw.any.tile < 0 || pw.M * pw.gk > 400000 || pw.gk * pw.gn > 400000) continue;
      g_case = sub + " " + tile + (compute == 2 ? " bf16x3" : compute ? " f32" : " f64") + (cplx ? " complex" : "");
      replay_plan(pw);
    }
  }
  unsetenv("SYMT_GEMM_TILE");
  for (int c = 0; c < 4 * n; ++c) {
    const int s = 1 + rng.below(3), t = 1 + rng.below(2), v = 1 + rng.below(2);
    const std::string L = "abcdefgh", I = L.substr(0, s), K = L.substr(s, v), J = L.substr(s + v, t);
    const std::string tu = rng.below(2) ? I + K : K + I, tv = rng.below(2) ? K + J : J + K, tw = rng.below(2) ? I + J : J + I;
    const int G = (int[]){4, 6, 8, 9, 12}[rng.below(5)];
    symt_group g{};
    g.nfactors = 1;
    g.order[0] = G;
    const bool cplx = rng.below(3) == 0;
    int32_t hs[8];
    int64_t dim[8];
    for (int m = 0; m < 8; ++m) {
      do hs[m] = 1 + rng.below(G); while (G % hs[m] != 0);
      if (rng.below(2)) hs[m] = G;
      dim[m] = 1 + rng.below(5);
    }
    struct Op { std::string sg; std::vector<int64_t> d; std::vector<int32_t> h; };
    auto desc = [&](const std::string& term, Op& o, bool second) {
      for (char m : term) {
        o.d.push_back(dim[m - 'a']);
        o.h.push_back(hs[m - 'a']);
        const bool neg = (m - 'a') % 2 == 1;
        o.sg.push_back((second && K.find(m) != std::string::npos ? !neg : neg) ? '-' : '+');
      }
      symt_tensor x{};
      x.nmodes = static_cast<int32_t>(term.size());
      x.signs = o.sg.c_str();
      x.charge = rng.below(G);
      x.dims = o.d.data();
      x.sectors = o.h.data();
      x.dtype = cplx ? SYMT_C128 : SYMT_F64;
      return x;
    };
    Op ou, ov;
    const symt_tensor u = desc(tu, ou, false), vv = desc(tv, ov, true);
    Plan p;
    std::string err;
    g_case = tu + "," + tv + "->" + tw + " sectors";
    if (make_plan((tu + "," + tv + "->" + tw).c_str(), &g, &u, &vv, nullptr, SYMT_COMPUTE_F64, &p, &err) != SYMT_OK) continue;
    check_workspace(p);
    if (p.direct) {
      check_workspace(*p.direct);
      check_direct(p);
    }
  }
  std::printf("%lld direct subgroup plans (%lld clear W)\n", static_cast<long long>(g_direct), static_cast<long long>(g_clear));
  std::printf("%lld checks, %lld plans (A along K %lld, K-major %lld, pairs %lld; complex V in place %lld; 4-byte "
              "only %lld; split-bf16 %lld), %lld K-step tails, %lld failures\n",
              static_cast<long long>(g_checks), static_cast<long long>(g_plans), static_cast<long long>(g_am[0]),
              static_cast<long long>(g_am[1]), static_cast<long long>(g_am[2]), static_cast<long long>(g_cb),
              static_cast<long long>(g_odd), static_cast<long long>(g_bf), static_cast<long long>(g_tails), static_cast<long long>(g_fail));
  return g_fail ? 1 : 0;
}
