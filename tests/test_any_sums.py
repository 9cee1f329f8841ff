"""The in-place product for any layout keeps binary32 sums short where it replaces a product
that cuts K: 128 indices each, then their sum."""
import sys

import pytest
import torch

from tests import planner as PL

DEV = "cuda:0"
K = 1024
# (subscripts, u's signs, |G|, rows, columns, operand type): taken by default, uncut by stream-K
CASES = [("ka,kb->ab", "-+", 6, 383, 628, torch.complex64), ("ak,kb->ab", "+-", 6, 177, 1267, torch.complex64),
         ("ka,kb->ab", "-+", 6, 432, 836, torch.float32), ("ak,kb->ab", "+-", 2, 356, 1300, torch.float32),
         ("ak,kb->ab", "+-", 6, 489, 912, torch.float32)]


def _u_dims(sub, M):
    return (M, K) if sub[0] == "a" else (K, M)


@pytest.mark.parametrize("case", CASES)
def test_planner_asks_for_short_sums(case):
    sub, su, G, M, N, dtype = case
    dt = PL.F32 if dtype == torch.float32 else PL.C64
    p, = PL.plans([PL.line(sub, (G,), su, _u_dims(sub, M), "++", (K, N), dt, "f32")])
    assert p["any"] >= 0 and p["chunk"] == 1 and p["sk"] == 0


def test_planner_keeps_the_other_sums():
    # binary64, and a binary32 product that cuts no K
    p = PL.plans([PL.line("ak,kb->ab", (9,), "+-", (500, 500), "++", (500, 500), PL.F64, "f64"),
                  PL.line("abcd,cdij->abij", (8,), "++--", (24, 24, 24, 24), "++--", (24, 24, 6, 6), PL.F32, "f32")])
    assert all(x["any"] >= 0 and x["chunk"] == 0 for x in p)


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_small_terms_of_a_long_sum_survive(case, monkeypatch):
    import paper_2007_08056_amd as P
    from paper_2007_08056_amd import symtensor as S

    sub, su, G, M, N, dtype = case
    for var in S._TUNING_VARS:
        monkeypatch.delenv(var, raising=False)
    # 1024 terms of 1 + 2^-17: every partial sum of 128, in any order, is exact in binary32, and
    # so is every sum of those; one sum past 512 has its last bit at 2^-14 and loses the 2^-17
    u = P.SymTensor(torch.ones((G,) + _u_dims(sub, M), dtype=dtype, device=DEV), su, 0, (G,))
    v = P.SymTensor(torch.full((G, K, N), 1 + 2.0 ** -17, dtype=dtype, device=DEV), "++", 0, (G,))
    for steps in (False, True):
        print(f"any sums {sub} G={G} {M} x {N} {dtype} steps={steps}", file=sys.stderr, flush=True)
        w = P.output_like(sub, u, v, dtype=dtype)
        w.data.fill_(float("nan"))
        P.contract_into(sub, u, v, w, "f32", steps=steps)
        assert w.data.eq(K * (1 + 2.0 ** -17)).all()
