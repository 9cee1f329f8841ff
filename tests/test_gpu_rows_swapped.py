"""The row-streaming product with its long side along N (a small matrix times a large tensor).

M and K at most 64, N long: the transposed product, rows along the columns of V and
W.  Forced on small shapes at the edges of its row blocks (32 binary64 or 64 binary32
rows): runs of contiguous columns shorter than, equal to and past a block, odd runs
(16-byte accesses at any element alignment), columns that are not contiguous in V or
in W (the general kernel), V starting one element into a buffer.  Against the
loop-over-blocks oracle (the product's bound) and bit for bit against the three-step
path, which runs the same product on the aligned forms.
"""
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
    ("ab,bcd->acd", (3,), "++", "-+-", (5, 7), (7, 5, 13)),            # runs of 65
    ("ab,bcd->acd", (2, 2), "+-", "++-", (57, 57), (57, 3, 19)),       # runs of 57, K and M of four tiles
    ("ab,bc->ac", (2,), "+-", "+-", (16, 4), (4, 128)),                # whole blocks
    ("ab,bc->ac", (5,), "+-", "+-", (1, 1), (1, 129)),                 # smallest M and K
    ("ba,bcd->cad", (3,), "+-", "-++", (17, 9), (17, 11, 8)),          # A K-major, W's columns split
    ("ab,cbd->adc", (3,), "++", "+--", (33, 31), (12, 31, 9)),         # V's contracted mode inside, W transposed
    ("abk,kcd->abcd", (2,), "++-", "+-+", (4, 4, 64), (64, 7, 31)),    # two output modes of U
]


@pytest.fixture(scope="module")
def P():
    import paper_2007_08056_amd as p
    return p


@pytest.mark.parametrize("compute", ["f64", "f32"])
@pytest.mark.parametrize("case", CASES)
def test_rows_along_n(P, case, compute, monkeypatch):
    sub, orders, cu, cv, du, dv = case
    monkeypatch.setenv("SYMT_GEMM_TILE", "rows")
    monkeypatch.delenv("SYMT_GEMM_SK", raising=False)
    rng = np.random.default_rng(seed("rows along n", sub, orders, du))
    g = O.Group(orders)
    su = O.Sym.make(cu, int(rng.integers(g.size)), du, g)
    sv = O.Sym.make(cv, int(rng.integers(g.size)), dv, g)
    dtype = torch.float64 if compute == "f64" else torch.float32
    u, v = (P.SymTensor(torch.from_numpy(rng.standard_normal(s.reduced_shape())).to(DEV, dtype), s.sign_string(),
                        s.charge, orders) for s in (su, sv))
    info = P.plan(sub, u, v, compute)
    print(f"rows along n {sub} {compute} M={info.m} K={info.k} N={info.n}", file=sys.stderr, flush=True)
    assert info.m <= 64 < info.n and info.k <= 64
    Ru, Rv = H.to_np(u.data).astype(np.float64), H.to_np(v.data).astype(np.float64)
    ref, _ = O.contract_blocks(sub, Ru, su, Rv, sv)
    absref, _ = O.contract_blocks(sub, np.abs(Ru), su, np.abs(Rv), sv)
    fac = H.bound_factor(compute, H.contracted_extent(sub, su))
    buf = torch.zeros(v.data.numel() + 1, dtype=dtype, device=DEV)
    buf[1:] = v.data.reshape(-1)
    v_off = P.SymTensor(buf[1:].view(v.data.shape), v.signs, v.charge, v.group)
    outs = []
    for vv, steps in ((v, False), (v, True), (v_off, False)):
        w = P.output_like(sub, u, v, dtype=dtype)
        w.data.fill_(float("nan"))
        P.contract_into(sub, u, vv, w, compute, steps=steps)
        assert np.all(np.abs(H.to_np(w.data).astype(np.float64) - ref) <= fac * absref + 1e-300)
        outs.append(w.data)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
