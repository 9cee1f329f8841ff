"""The long-K product's vector variant (csrc/gemm_tallk.hip): operands whose runs along K
are long but not whole 16-byte chunks, groups that cross a run's end or K's end, clamped
last chunks of B's rows.

Checked against the loop-over-blocks oracle and bit for bit against the three-step path
(the same groups of K in the same order, also on the vector variant) and the same
contraction with U and V starting one element into a buffer.
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
    # (subscripts, group, signs of u and v, dims of u, dims of v): M, N and runs of K
    ("abc,bcd->ad", (2,), "+--", "++-", (57, 23, 25), (23, 25, 57)),        # odd M, N; runs of 575
    ("ab,bc->ac", (3,), "+-", "+-", (1, 1031), (1031, 5)),                  # one row; N one past a chunk; K tail
    ("abc,bcd->ad", (2, 2), "+--", "++-", (17, 257, 1), (257, 1, 33)),      # runs of 257: groups cross them often
    ("abc,cd->abd", (2,), "++-", "+-", (5, 3, 2051), (2051, 15)),           # two row modes (A from its start)
    ("ab,bcd->acd", (2,), "+-", "+--", (31, 1201), (1201, 4, 7)),           # two column modes, runs of 28
    ("ab,bcd->acd", (3,), "+-", "+--", (20, 1025), (1025, 4, 5)),           # columns in runs of 20: chunks
    ("abc,bcd->ad", (2,), "+--", "++-", (64, 16, 67), (16, 67, 64)),        # whole tiles, runs of 1072
]


@pytest.fixture(scope="module")
def P():
    import paper_2007_08056_amd as p
    return p


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("case", CASES)
def test_long_k_vector_variant(P, case, dtype, monkeypatch):
    sub, orders, cu, cv, du, dv = case
    monkeypatch.setenv("SYMT_GEMM_TILE", "tallk")
    rng = np.random.default_rng(seed("tallk-vec", sub, orders, str(du)))
    g = O.Group(orders)
    su = O.Sym.make(cu, int(rng.integers(g.size)), du, g)
    sv = O.Sym.make(cv, int(rng.integers(g.size)), dv, g)
    print(f"long K {sub} G={orders} {dtype} {du} {dv}", file=sys.stderr, flush=True)
    compute = "f64" if dtype == torch.float64 else "f32"

    def draw(sym):
        x = torch.from_numpy(rng.standard_normal(sym.reduced_shape())).to(DEV, dtype)
        return P.SymTensor(x, sym.sign_string(), sym.charge, orders)

    def off(x):
        buf = torch.full((x.data.numel() + 2,), float("nan"), dtype=dtype, device=DEV)
        buf[1:-1] = x.data.reshape(-1)
        return P.SymTensor(buf[1:-1].view(x.data.shape), x.signs, x.charge, x.group)
    u, v = draw(su), draw(sv)
    Ru, Rv = H.to_np(u.data).astype(np.float64), H.to_np(v.data).astype(np.float64)
    ref, _ = O.contract_blocks(sub, Ru, su, Rv, sv)
    absref, _ = O.contract_blocks(sub, np.abs(Ru), su, np.abs(Rv), sv)
    fac = H.bound_factor(compute, H.contracted_extent(sub, su))
    outs = []
    for uu, vv, steps in ((u, v, False), (off(u), off(v), False), (u, v, True)):
        w = P.output_like(sub, u, v, dtype=dtype)
        w.data.fill_(float("nan"))
        P.contract_into(sub, uu, vv, w, compute, steps=steps)
        outs.append(w.data)
    assert np.all(np.abs(H.to_np(outs[0]).astype(np.float64) - ref) <= fac * absref + 1e-300)
    assert torch.equal(outs[0], outs[1])
    assert torch.equal(outs[0], outs[2])
