"""Workspace sizes of planned contractions (host only)."""
import random

import pytest
import torch

import paper_2007_08056_amd as P

FORMS = [("abkl,klij->abij", "++--", "++--"), ("klab,klij->abij", "--++", "++--"), ("ak,kb->ab", "+-", "+-"),
         ("abk,ki->abi", "++-", "+-"), ("ka,kb->ab", "-+", "+-")]


def _contraction(rng, dtype, forms=FORMS):
    """Random operands of one contraction, as shapes alone."""
    G = rng.choice([2, 3, 4, 6, 8])
    sub, su, sv = rng.choice(forms)
    tu, tv = sub.split("->")[0].split(",")
    tw = sub.split("->")[1]
    d = {c: rng.choice([rng.randint(1, 12), 4 * rng.randint(1, 10), rng.randint(1, 64)]) for c in tu + tv}

    def make(term, signs, charge=0):
        return P.SymTensor(torch.empty([G] * (len(term) - 1) + [d[c] for c in term], dtype=dtype, device="meta"), signs,
                           charge, (G,))
    u, v = make(tu, su), make(tv, sv)
    return sub, u, v, lambda info: make(tw, info.w_signs.decode(), info.w_charge)


@pytest.mark.parametrize("dtype,compute", [(torch.float64, "f64"), (torch.float32, "f32"), (torch.float32, "bf16x3"),
                                           (torch.complex128, "f64"), (torch.complex64, "f32")])
def test_a_workspace_planned_without_w_serves_a_w_of_the_compute_type(dtype, compute, monkeypatch):
    monkeypatch.delenv("SYMT_GEMM_TILE", raising=False)
    rng = random.Random(20070805)
    for _ in range(400):
        sub, u, v, out = _contraction(rng, dtype)
        info = P.plan(sub, u, v, compute)
        w = out(info)
        assert P.plan(sub, u, v, compute, w=w).workspace_bytes <= info.workspace_bytes, (sub, u.group, u.dims, v.dims)
