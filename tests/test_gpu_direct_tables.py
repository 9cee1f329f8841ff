"""A contraction whose split-bf16 product depends on U's alignment (256-row stream-K tiles
that read U in place where it is 16-byte aligned, the replaced product elsewhere): each of
the two keeps offset tables of its own, whichever alignment the first call has."""
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
    # (subscripts, |G|, signs, dims of u and v, forced tile): the replaced product aligns U in
    # all (affine tables of U_al, as many bytes as U's own)
    ("abcd,cdij->abij", 3, "++--", "++--", (28, 28, 24, 24), (24, 24, 14, 14), None),
    ("abcd,cdij->abij", 8, "++--", "++--", (11, 11, 18, 8), (18, 8, 9, 9), None),
    ("abcd,cdij->abij", 8, "++--", "++--", (6, 6, 4, 4), (4, 4, 4, 9), "bw256x288sk"),
]


@pytest.mark.parametrize("order", [(1, 0, 1), (0, 1, 0)])
@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_tables_of_aligned_and_unaligned_u(case, prepared, order, monkeypatch):
    import ctypes

    import paper_2007_08056_amd as P
    from paper_2007_08056_amd import _lib as L
    from paper_2007_08056_amd import symtensor as S

    sub, G, cu, cv, du, dv, tile = case
    for var in S._TUNING_VARS:
        monkeypatch.delenv(var, raising=False)
    if tile:
        monkeypatch.setenv("SYMT_GEMM_TILE", tile)
    rng = np.random.default_rng(seed("direct-tables", sub, (G,)))
    g = O.Group((G,))
    # (a charge of its own per variant: a plan that no other call has used yet)
    su = O.Sym.make(cu, order[0], du, g)
    sv = O.Sym.make(cv, 2 if prepared else 1, dv, g)
    print(f"direct tables {sub} G={G} {tile} prepared={prepared} {order}", file=sys.stderr, flush=True)

    def draw(sym):
        x = torch.from_numpy(rng.standard_normal(sym.reduced_shape())).to(DEV, torch.float32)
        return P.SymTensor(x, sym.sign_string(), sym.charge, (G,))
    u, v = draw(su), draw(sv)
    Ru, Rv = H.to_np(u.data).astype(np.float64), H.to_np(v.data).astype(np.float64)
    ref, _ = O.contract_blocks(sub, Ru, su, Rv, sv)
    absref, _ = O.contract_blocks(sub, np.abs(Ru), su, np.abs(Rv), sv)
    fac = H.bound_factor("bf16x3", H.contracted_extent(sub, su)) + H.U32
    buf = torch.zeros(u.data.numel() + 1, dtype=torch.float32, device=DEV)
    buf[1:] = u.data.reshape(-1)
    off = P.SymTensor(buf[1:].view(u.data.shape), u.signs, u.charge, u.group)
    w = P.output_like(sub, u, v)
    ws = torch.empty(max(1, P.plan(sub, u, v, "bf16x3", w=w).workspace_bytes), dtype=torch.uint8, device=DEV)
    grp, dg, dw = L.make_group((G,)), v.desc(), w.desc()
    for unaligned in order:
        x = off if unaligned else u
        w.data.fill_(float("nan"))
        if prepared:
            P.contract_into(sub, x, v, w, "bf16x3", ws)
        else:
            L.check(L.LIB.symtensor_contract(L.context(0), sub.encode(), ctypes.byref(grp), x.desc().ref, dg.ref, dw.ref,
                                             L.COMPUTE["bf16x3"], ctypes.c_void_p(ws.data_ptr()), ws.numel(),
                                             ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)), L.context(0))
        off_by = np.abs(H.to_np(w.data).astype(np.float64) - ref) - fac * absref
        assert not off_by.max() > 1e-300 and not np.isnan(off_by).any(), unaligned
