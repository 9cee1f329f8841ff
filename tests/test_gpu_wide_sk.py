"""The split-bf16 product on 256 x (192 to 288) tiles under stream-K (csrc/gemm_bf16x3.hip):
M and N ragged against the tiles, cut and whole tiles, W in binary32 and binary64; bit for
bit the three-step path on the same tiles, and within the product's bound of the oracle."""
import sys

import numpy as np
import pytest
import torch

import oracle as O
from tests import gpu_helpers as H
from tests.seeding import seed

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # (subscripts, group, signs, dims of u and v)
    ("abcd,cdij->abij", (8,), "++--", "++--", (6, 6, 8, 8), (8, 8, 4, 9)),      # 288 x 512 x 288, cut tiles
    ("abcd,cdij->abij", (2, 4), "++--", "++--", (5, 7, 4, 4), (4, 4, 5, 5)),    # 280 x 128 x 200, runs of 16
    ("ak,kb->ab", (3,), "+-", "++", (513, 96), (96, 195)),                      # three K-steps a tile
]


@pytest.fixture(scope="module")
def P():
    import paper_2007_08056_amd as p
    return p


@pytest.mark.parametrize("bn", [192, 224, 256, 288])
@pytest.mark.parametrize("case", CASES)
def test_wide_stream_k_split_bf16(P, case, bn, monkeypatch):
    sub, orders, cu, cv, du, dv = case
    monkeypatch.setenv("SYMT_GEMM_TILE", f"bw256x{bn}sk")
    monkeypatch.delenv("SYMT_GEMM_SK", raising=False)
    monkeypatch.delenv("SYMT_BF16_FA", raising=False)
    rng = np.random.default_rng(seed("wide-sk", sub, orders))
    g = O.Group(orders)
    su = O.Sym.make(cu, int(rng.integers(g.size)), du, g)
    sv = O.Sym.make(cv, int(rng.integers(g.size)), dv, g)
    print(f"wide stream-K {sub} G={orders} 256x{bn}", file=sys.stderr, flush=True)

    def draw(sym):
        x = torch.from_numpy(rng.standard_normal(sym.reduced_shape())).to(DEV, torch.float32)
        return P.SymTensor(x, sym.sign_string(), sym.charge, orders)
    u, v = draw(su), draw(sv)
    Ru, Rv = H.to_np(u.data).astype(np.float64), H.to_np(v.data).astype(np.float64)
    ref, _ = O.contract_blocks(sub, Ru, su, Rv, sv)
    absref, _ = O.contract_blocks(sub, np.abs(Ru), su, np.abs(Rv), sv)
    fac = H.bound_factor("bf16x3", H.contracted_extent(sub, su))
    buf = torch.zeros(u.data.numel() + 1, dtype=torch.float32, device=DEV)
    buf[1:] = u.data.reshape(-1)
    u_off = P.SymTensor(buf[1:].view(u.data.shape), u.signs, u.charge, u.group)
    outs = []
    for uu, wt, steps in ((u, torch.float64, False), (u, torch.float64, True), (u, torch.float32, False),
                          (u, torch.float32, True), (u_off, torch.float64, False)):
        w = P.output_like(sub, u, v, dtype=wt)
        w.data.fill_(float("nan"))
        P.contract_into(sub, uu, v, w, "bf16x3", steps=steps)
        outs.append(w.data)
    for o in (outs[0], outs[4]):                 # (an unaligned U takes the other tiles)
        assert np.all(np.abs(H.to_np(o) - ref) <= fac * absref + 1e-300)
    assert torch.equal(outs[0], outs[1])
    assert torch.equal(outs[2], outs[0].to(torch.float32)) and torch.equal(outs[2], outs[3])
