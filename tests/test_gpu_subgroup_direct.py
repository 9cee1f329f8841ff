"""Subgroup contractions on their live slices in place (offset tables of the live slices,
W written in place, blocks of W that no slice reaches cleared), against the loop-over-blocks
oracle and the three-step path, over layouts, compute modes and W's order."""
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
    # (subscripts, |G|, signs, dims and sector counts of u and of v)
    ("abcd,cdij->abij", 8, "++--", "++--", (6, 6, 6, 6), (6, 6, 3, 4), (4, 4, 8, 8), (8, 8, 8, 8)),
    ("abcd,cdij->abij", 6, "++--", "++--", (9, 9, 5, 5), (5, 5, 3, 3), (3, 3, 6, 6), (6, 6, 6, 6)),      # odd runs of K
    ("ak,ki->ia", 8, "+-", "+-", (40, 33), (33, 29), (4, 8), (8, 8)),            # half of W's blocks not reached
    ("abk,ki->abi", 12, "++-", "+-", (5, 7, 24), (24, 50), (2, 4, 12), (12, 12)),   # last member solves for the others
    ("klab,klij->abij", 8, "--++", "++--", (4, 6, 8, 4), (4, 6, 4, 4), (8, 8, 4, 4), (8, 8, 8, 8)),      # K-major
    ("ak,ik->ai", 4, "+-", "-+", (20, 300), (17, 300), (2, 4), (4, 4)),          # V's contracted mode last
]


@pytest.fixture(scope="module")
def P():
    import paper_2007_08056_amd as p
    return p


@pytest.mark.parametrize("compute,dt", [("f64", torch.float64), ("f32", torch.float32), ("bf16x3", torch.float32),
                                        ("f64", torch.complex128), ("f32", torch.complex64)])
@pytest.mark.parametrize("case", CASES)
def test_subgroup_contraction_in_place(P, case, compute, dt, monkeypatch):
    sub, G, cu, cv, du, dv, hu, hv = case
    monkeypatch.delenv("SYMT_GEMM_TILE", raising=False)
    rng = np.random.default_rng(seed("subgroup-direct", sub, G))
    g = O.Group((G,))
    su = O.Sym.make(cu, 0, du, g, sectors=hu)
    sv = O.Sym.make(cv, 2, dv, g, sectors=hv)
    print(f"subgroup direct {sub} G={G} {hu} {hv} {compute}", file=sys.stderr, flush=True)
    cplx = dt.is_complex
    wide = np.complex128 if cplx else np.float64

    def draw(sym):
        x = rng.standard_normal(sym.reduced_shape())
        x = x + 1j * rng.standard_normal(x.shape) if cplx else x
        return P.SymTensor(torch.from_numpy(x).to(DEV, dt), sym.sign_string(), sym.charge, (G,), None, sym.sectors)
    u, v = draw(su), draw(sv)
    Ru, Rv = H.to_np(u.data).astype(wide), H.to_np(v.data).astype(wide)
    ref, sw = O.contract_blocks(sub, Ru, su, Rv, sv)
    absref, _ = O.contract_blocks(sub, np.abs(Ru), su, np.abs(Rv), sv)
    fac = H.bound_factor(compute, (2 if cplx else 1) * H.contracted_extent(sub, su)) + (H.U32 if compute == "bf16x3" else 0)
    assert P.plan(sub, u, v, compute).fused == 0
    for steps in (False, True):
        w = P.output_like(sub, u, v, dtype=dt)
        w.data.fill_(float("nan"))
        P.contract_into(sub, u, v, w, compute, steps=steps)
        got = H.to_np(w.data).astype(wide)
        for part in (np.real, np.imag):
            assert np.all(np.abs(part(got) - part(ref)) <= fac * absref + 1e-300), steps
        assert all(np.all(got[st] == 0) for st in H.dead_stored_tuples(sw))
