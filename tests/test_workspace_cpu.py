"""Workspace sizes of planned contractions (host only)."""
import random

import pytest
import torch

import paper_2007_08056_amd as P
from tests import planner as PL

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


def test_pieces_are_sized_by_the_work_that_can_be_cut():
    # (product, largest workspace in MB): 50.4 and 25 MB were reserved for these
    cases = [(PL.line("ak,kb->ab", (5,), "+-", (120, 320), "++", (320, 90), PL.F32, "bf16x3"), 8),
             (PL.line("abkl,klij->abij", (3,), "++--", (2, 40, 38, 5), "++--", (38, 5, 16, 2), PL.C64, "f32"), 14)]
    for (ln, most), p in zip(cases, PL.plans([ln for ln, _ in cases])):
        assert p["any"] >= 0 and p["workspace"] <= most << 20, p
    # two pieces per workgroup of at least four K-steps each
    rng = random.Random(3)
    lines, info = [], []
    for _ in range(1500):
        sub, su = rng.choice([("ak,kb->ab", "+-"), ("ka,kb->ab", "-+")])
        G, M, N, K = rng.choice([1, 2, 4, 8]), rng.randint(1, 1500), rng.randint(1, 1500), rng.randint(1, 3000)
        dt, comp = rng.choice([(PL.F64, "f64"), (PL.F32, "f32"), (PL.C64, "f32"), (PL.F32, "bf16x3")])
        lines.append(PL.line(sub, (G,), su, (M, K) if sub[0] == "a" else (K, M), "++", (K, N), dt, comp))
        info.append((comp, 8 if comp != "f32" else 4))
    cut = 0
    for (comp, piece), p in zip(info, PL.plans(lines)):
        if p["any"] < 0 or not p["sk"] or p["wide_bn"]:
            continue
        tiles = [(128, 128) if comp == "bf16x3" else (96, 96), (128, 64), (64, 64)]
        steps = -(-p["k"] // (16 if comp == "f64" else 32))
        most = 0
        for bm, bn in {tiles[p["any"]], tiles[max(p["any"], 1)]}:
            work = p["nq"] * -(-p["m"] // bm) * -(-p["n"] // bn) * steps
            most = max(most, 2 * (work // 4) * bm * bn * piece)
        assert p["partial"] <= most, p
        cut += p["partial"] > 0
    assert cut > 100
