// Prints what the planner takes for contractions read from standard input, one per line:
//   einsum factors(a,b,..) u_signs u_charge u_dims u_sectors v_signs v_charge v_dims v_sectors u_dtype v_dtype w_dtype compute
// (lists comma-separated, "-" for none; dtypes and compute as in symtensor.h, compute | 0x100 = three steps;
// w_dtype -1: no w).  One line of key=value pairs each.
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "plan.hpp"

using namespace symt;

template <typename T>
static std::vector<T> list(const std::string& s) {
  std::vector<T> out;
  if (s == "-") return out;
  std::stringstream ss(s);
  std::string x;
  while (std::getline(ss, x, ',')) out.push_back(static_cast<T>(std::stoll(x)));
  return out;
}

int main() {
  std::string line;
  while (std::getline(std::cin, line)) {
    std::stringstream in(line);
    std::string einsum, fac, us, ud, uh, vs, vd, vh;
    int uc, vc, udt, vdt, wdt, compute;
    if (!(in >> einsum >> fac >> us >> uc >> ud >> uh >> vs >> vc >> vd >> vh >> udt >> vdt >> wdt >> compute)) return 2;
    symt_group g{};
    for (int f : list<int>(fac)) g.order[g.nfactors++] = f;
    auto dims_u = list<int64_t>(ud), dims_v = list<int64_t>(vd);
    auto sec_u = list<int32_t>(uh), sec_v = list<int32_t>(vh);
    auto desc = [](const std::string& sg, int c, std::vector<int64_t>& d, std::vector<int32_t>& h, int dt) {
      symt_tensor x{};
      x.nmodes = static_cast<int32_t>(d.size());
      x.signs = sg.c_str();
      x.charge = c;
      x.dims = d.data();
      x.dtype = dt;
      x.sectors = h.empty() ? nullptr : h.data();
      return x;
    };
    const symt_tensor u = desc(us, uc, dims_u, sec_u, udt), v = desc(vs, vc, dims_v, sec_v, vdt);
    Plan p;
    std::string err;
    int rc = make_plan(einsum.c_str(), &g, &u, &v, nullptr, compute, &p, &err);
    if (rc == SYMT_OK && wdt >= 0) {
      std::string sw;
      std::vector<int64_t> dw(p.W.dims, p.W.dims + p.W.n);
      std::vector<int32_t> hw;
      if (!sec_u.empty() || !sec_v.empty()) hw.assign(p.W.hs, p.W.hs + p.W.n);
      for (int m = 0; m < p.W.n; ++m) sw.push_back(p.w_sign[m] > 0 ? '+' : '-');
      const symt_tensor w = desc(sw, p.w_charge, dw, hw, wdt);
      Plan q;
      rc = make_plan(einsum.c_str(), &g, &u, &v, &w, compute, &q, &err);
      p = q;
    }
    if (rc != SYMT_OK) {
      std::printf("error=%d\n", rc);
      continue;
    }
    const Plan& d = p.direct ? *p.direct : p;
    const GemmChoice c = p.compute == SYMT_COMPUTE_BF16X3
                             ? GemmChoice{}
                             : choose_fp_gemm(d.nq, d.M, d.gn, d.gk, p.compute == SYMT_COMPUTE_F64 ? 8 : 4, true, d.a_trans, d.long_cols);
    std::printf("fused=%d fused_ua=%d any=%d am=%d ch16=%d sk=%d chunk=%d cb=%d any_direct=%d direct=%d slices=%d wide_bn=%d "
                "tile=%d splits=%d tile_sk=%d workspace=%zu partial=%zu nq=%lld m=%lld k=%lld n=%lld\n",
                p.fused, p.fused_ua, d.any.tile, d.any.am, d.any.ch16, d.any.sk, d.any.chunk, d.any.cb, d.any_direct, p.direct != nullptr,
                d.slices, d.wide_bn, c.tile, c.splits, c.sk, p.workspace, d.bytes_partial, static_cast<long long>(d.nq),
                static_cast<long long>(d.M), static_cast<long long>(d.gk), static_cast<long long>(d.gn));
  }
  return 0;
}
