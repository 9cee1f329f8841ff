"""The 256-row split-bf16 tiles under stream-K keep the cross terms' sum apart from the
hi hi sum and join the two in binary64: terms below the larger sum's last bit are kept."""
import sys

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("bn", [192, 224, 256, 288])
@pytest.mark.parametrize("steps", [False, True])
def test_small_cross_terms_survive(bn, steps, monkeypatch):
    import paper_2007_08056_amd as P

    monkeypatch.setenv("SYMT_GEMM_TILE", f"bw256x{bn}sk")
    for var in ("SYMT_GEMM_SK", "SYMT_BF16_FA"):
        monkeypatch.delenv(var, raising=False)
    K = 4800
    print(f"wide sums 256x{bn} steps={steps}", file=sys.stderr, flush=True)
    # u = 1 + 2^-17: hi = 1, lo = 2^-17.  The hi hi sum (up to 4800) and the cross sum (up to
    # 4800 2^-17) are exact in binary32 each; a common sum past 4096 has its last bit at 2^-11
    # and loses a 32-deep step's 2^-12
    u = P.SymTensor(torch.full((2, 513, K), 1 + 2.0 ** -17, device=DEV), "+-", 0, (2,))
    v = P.SymTensor(torch.ones(2, K, 300, device=DEV), "++", 0, (2,))
    for dtype in (torch.float64, torch.float32):
        w = P.output_like("ak,kb->ab", u, v, dtype=dtype)
        w.data.fill_(float("nan"))
        P.contract_into("ak,kb->ab", u, v, w, "bf16x3", steps=steps)
        want = torch.tensor(K * (1 + 2.0 ** -17), dtype=torch.float64).to(dtype).item()
        assert w.data.eq(want).all(), (w.data.min().item(), w.data.max().item(), want)
