"""The in-place product for any layout and the three-step path give the same bits by default,
also where the two load their operands with different widths or run under stream-K."""
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
    # (subscripts, |G|, signs and dims of u and v, operand type, compute)
    ("abcd,cdij->abij", 8, "++--", (25, 9, 15, 20), "++--", (15, 20, 3, 3), torch.float64, "f64"),   # chunks in U_al only
    ("abcd,cdij->abij", 8, "++--", (3, 4, 16, 14), "++--", (16, 14, 29, 6), torch.float32, "f32"),
    ("ka,kb->ab", 4, "-+", (1493, 800), "++", (1493, 452), torch.float64, "f64"),                    # chunks in U only
    ("ka,kb->ab", 3, "-+", (1307, 552), "++", (1307, 188), torch.complex64, "f32"),
    ("ka,kb->ab", 2, "-+", (1254, 508), "++", (1254, 496), torch.float32, "bf16x3"),
    ("ka,kb->ab", 1, "-+", (766, 412), "++", (766, 224), torch.float32, "bf16x3"),
]


@pytest.mark.parametrize("case", CASES)
def test_steps_and_in_place_sum_alike(case, monkeypatch):
    import paper_2007_08056_amd as P
    from paper_2007_08056_amd import symtensor as S

    sub, G, cu, du, cv, dv, dtype, compute = case
    for var in S._TUNING_VARS:
        monkeypatch.delenv(var, raising=False)
    rng = np.random.default_rng(seed("any-steps", sub, (G,)))
    g = O.Group((G,))
    su, sv = O.Sym.make(cu, 0, du, g), O.Sym.make(cv, 0, dv, g)
    print(f"any steps {sub} G={G} {du} {dv} {dtype}", file=sys.stderr, flush=True)
    wide = np.complex128 if dtype.is_complex else np.float64

    def draw(sym):
        x = rng.standard_normal(sym.reduced_shape())
        x = x + 1j * rng.standard_normal(x.shape) if dtype.is_complex else x
        return P.SymTensor(torch.from_numpy(x).to(DEV, dtype), sym.sign_string(), sym.charge, (G,))
    u, v = draw(su), draw(sv)
    Ru, Rv = H.to_np(u.data).astype(wide), H.to_np(v.data).astype(wide)
    ref, _ = O.contract_blocks(sub, Ru, su, Rv, sv)
    absref, _ = O.contract_blocks(sub, np.abs(Ru), su, np.abs(Rv), sv)
    fac = H.bound_factor(compute, (2 if dtype.is_complex else 1) * H.contracted_extent(sub, su)) + (H.U32 if compute == "bf16x3" else 0)
    outs = []
    for steps in (False, True):
        w = P.output_like(sub, u, v, dtype=dtype)
        w.data.fill_(float("nan"))
        P.contract_into(sub, u, v, w, compute, steps=steps)
        got = H.to_np(w.data).astype(wide)
        for part in (np.real, np.imag):
            worst = (np.abs(part(got) - part(ref)) - fac * absref).max()
            assert worst <= 1e-300, steps
        outs.append(w.data)
    assert torch.equal(outs[0], outs[1])
