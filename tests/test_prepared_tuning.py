"""A prepared contraction runs as it was planned, whatever the tuning variables hold later."""
import pytest
import torch

import paper_2007_08056_amd as P
from paper_2007_08056_amd import _lib as L
from paper_2007_08056_amd import symtensor as S

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (G, rows, K, columns, type, compute, variables at planning, variables at the run)
CASES = [
    (2, 520, 64, 300, torch.float32, "bf16x3", {"SYMT_GEMM_TILE": "bw256x256s2"}, {}),      # interleaved planes
    (2, 520, 64, 300, torch.float32, "bf16x3", {"SYMT_GEMM_TILE": "b128x128k32"}, {"SYMT_GEMM_TILE": "bd256x128s3"}),
    (2, 520, 64, 300, torch.float32, "bf16x3", {}, {"SYMT_GEMM_TILE": "bw256x128s3", "SYMT_BF16_IL": "0"}),
    (3, 200, 1000, 190, torch.float64, "f64", {}, {"SYMT_GEMM_TILE": "128x48", "SYMT_GEMM_SK": "0"}),
    (3, 200, 1000, 190, torch.float32, "f32", {"SYMT_GEMM_TILE": "64x96"}, {"SYMT_GEMM_SK": "0"}),
    (3, 60, 4096, 50, torch.float32, "f32", {}, {"SYMT_GEMM_SK": "0"}),                     # the long-K product
    (3, 200, 1000, 190, torch.float64, "f64", {"SYMT_FUSED_V": "0"}, {"SYMT_GEMM_TILE": "d96x96s2"}),
]


@pytest.mark.parametrize("case", CASES)
def test_runs_keep_the_plan_of_their_handle(case, monkeypatch):
    G, M, K, N, dtype, compute, before, after = case
    for var in S._TUNING_VARS:
        monkeypatch.delenv(var, raising=False)
    g = torch.Generator().manual_seed(M + K)
    u = P.SymTensor(torch.randn(G, M, K, generator=g, dtype=torch.float64).to(DEV, dtype), "+-", 0, (G,))
    v = P.SymTensor(torch.randn(G, K, N, generator=g, dtype=torch.float64).to(DEV, dtype), "++", 0, (G,))
    w = P.output_like("ak,kb->ab", u, v, dtype=dtype)
    for k, x in before.items():
        monkeypatch.setenv(k, x)
    need = P.plan("ak,kb->ab", u, v, compute, w=w).workspace_bytes
    h = L.Prepared(0, "ak,kb->ab", L.make_group((G,)), u.desc(), v.desc(), w.desc(), S._code(compute, False))
    ws = torch.empty(max(1, need), dtype=torch.uint8, device=DEV)

    def run():
        w.data.fill_(float("nan"))
        h.run(u.data.data_ptr(), v.data.data_ptr(), w.data.data_ptr(), ws.data_ptr(), need,
              torch.cuda.current_stream().cuda_stream)
        return w.data.clone()
    want = run()
    exact = torch.bmm(u.data.double(), v.data.double())
    assert (want.double() - exact).abs().max() <= (1e-3 if dtype == torch.float32 else 1e-10) * K ** .5
    for var in before:
        monkeypatch.delenv(var)
    for k, x in after.items():
        monkeypatch.setenv(k, x)
    assert torch.equal(run(), want)
