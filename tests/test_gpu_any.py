"""The in-place product for any layout (csrc/gemm_any.hpp) at the edges of its tiles and loads.

Each of its tiles is forced on small ragged contractions: odd block sizes (4-byte
loads), K runs shorter than, equal to and past a K-step, U's contracted modes last,
first and in between, real and complex, stream-K on and off, and U starting one
element into a buffer.  Checked against the loop-over-blocks oracle element by
element (the product's bound) and bit for bit against the three-step path, which
multiplies the aligned forms on the same tile.
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
    # (subscripts, group, signs of u and v, dims of u, dims of v)
    ("abkl,klij->abij", (4,), "++--", "++--", (3, 5, 4, 4), (4, 4, 2, 3)),        # runs of one f64 step, half an f32 one
    ("ak,kb->ab", (2, 3), "+-", "++", (65, 33), (33, 97)),                         # odd, one past a K-step and a tile
    ("ak,kb->ba", (2,), "+-", "+-", (96, 500), (500, 64)),                         # whole tiles, K tail, W transposed
    ("abkl,klij->abij", (3,), "++--", "++--", (7, 3, 3, 5), (3, 5, 5, 7)),         # odd runs of 15
    ("klab,klij->abij", (4,), "--++", "++--", (4, 8, 3, 6), (4, 8, 2, 6)),         # K-major, whole chunks
    ("opij,opkm->ijmk", (2, 2), "++--", "--++", (3, 5, 3, 3), (3, 5, 4, 5)),       # K-major, odd, W's columns transposed
    ("akbl,klij->abij", (3,), "+-+-", "++--", (4, 3, 6, 5), (3, 5, 4, 2)),         # contracted modes in between
    ("abk,ijk->abij", (3,), "++-", "--+", (5, 4, 9), (6, 5, 9)),                   # V's contracted mode last: V aligned
]


@pytest.fixture(scope="module")
def P():
    import paper_2007_08056_amd as p
    return p


@pytest.mark.parametrize("tile", ["a96x96s2", "a128x64s2", "a64x64s2"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.complex128, torch.complex64])
@pytest.mark.parametrize("case", CASES)
def test_any_layout_product(P, case, dtype, tile, monkeypatch):
    sub, orders, cu, cv, du, dv = case
    monkeypatch.setenv("SYMT_GEMM_TILE", tile)
    rng = np.random.default_rng(seed("any", sub, orders))
    g = O.Group(orders)
    su = O.Sym.make(cu, int(rng.integers(g.size)), du, g)
    sv = O.Sym.make(cv, int(rng.integers(g.size)), dv, g)
    print(f"any {sub} G={orders} {dtype} {tile}", file=sys.stderr, flush=True)
    cplx = dtype.is_complex
    compute = "f64" if dtype in (torch.float64, torch.complex128) else "f32"

    def draw(sym):
        x = rng.standard_normal(sym.reduced_shape())
        x = x + 1j * rng.standard_normal(x.shape) if cplx else x
        return P.SymTensor(torch.from_numpy(x).to(DEV, dtype), sym.sign_string(), sym.charge, orders)
    u, v = draw(su), draw(sv)
    wide = np.complex128 if cplx else np.float64
    Ru, Rv = H.to_np(u.data).astype(wide), H.to_np(v.data).astype(wide)
    ref, _ = O.contract_blocks(sub, Ru, su, Rv, sv)
    absref, _ = O.contract_blocks(sub, np.abs(Ru), su, np.abs(Rv), sv)
    fac = H.bound_factor(compute, (2 if cplx else 1) * H.contracted_extent(sub, su))

    def check(w):
        got = H.to_np(w.data).astype(wide)
        for part in (np.real, np.imag) if cplx else (np.asarray,):
            assert np.all(np.abs(part(got) - part(ref)) <= fac * absref + 1e-300)
    buf = torch.zeros(u.data.numel() + 1, dtype=dtype, device=DEV)
    buf[1:] = u.data.reshape(-1)
    u_off = P.SymTensor(buf[1:].view(u.data.shape), u.signs, u.charge, u.group)
    for sk in ("0", "1"):
        monkeypatch.setenv("SYMT_GEMM_SK", sk)
        outs = []
        for uu, steps in ((u, False), (u, True), (u_off, False)):
            w = P.output_like(sub, u, v, dtype=dtype)
            w.data.fill_(float("nan"))
            P.contract_into(sub, uu, v, w, compute, steps=steps)
            check(w)
            outs.append(w.data)
        assert torch.equal(outs[0], outs[2])        # the loads' width does not change the sums
        assert torch.equal(outs[0], outs[1])        # nor does aligning the operands first


@pytest.mark.parametrize("tile", ["a128x128s2", "a128x64s2", "a64x64s2"])
@pytest.mark.parametrize("case", CASES)
def test_any_layout_split_bf16_product(P, case, tile, monkeypatch):
    """Split-bf16 on binary32 operands, split as the fragments are read: W in binary32
    and in binary64 (the same sums), three steps and an odd U the same bits."""
    sub, orders, cu, cv, du, dv = case
    monkeypatch.setenv("SYMT_GEMM_TILE", tile)
    rng = np.random.default_rng(seed("any-bf16", sub, orders))
    g = O.Group(orders)
    su = O.Sym.make(cu, int(rng.integers(g.size)), du, g)
    sv = O.Sym.make(cv, int(rng.integers(g.size)), dv, g)
    print(f"any split-bf16 {sub} G={orders} {tile}", file=sys.stderr, flush=True)

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
    for sk in ("0", "1"):
        monkeypatch.setenv("SYMT_GEMM_SK", sk)
        outs = []
        for uu, wt, steps in ((u, torch.float64, False), (u, torch.float64, True), (u_off, torch.float64, False),
                              (u, torch.float32, False), (u, torch.float32, True)):
            w = P.output_like(sub, u, v, dtype=wt)
            w.data.fill_(float("nan"))
            P.contract_into(sub, uu, v, w, "bf16x3", steps=steps)
            outs.append(w.data)
        assert np.all(np.abs(H.to_np(outs[0]) - ref) <= fac * absref + 1e-300)
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
        assert torch.equal(outs[3], outs[0].to(torch.float32)) and torch.equal(outs[3], outs[4])
