"""What einsum checks of its operands' data, forward and backward."""
import pytest
import torch

import paper_2007_08056_amd as P
from paper_2007_08056_amd import symtensor as S

SUB = "abkl,klij->abij"


@pytest.mark.parametrize("operand", [0, 1])
@pytest.mark.parametrize("device", ["cpu", pytest.param("cuda:0", marks=pytest.mark.gpu)])
def test_data_set_to_other_sector_extents_is_refused(operand, device):
    make = lambda: P.SymTensor(torch.zeros(4, 4, 4, 2, 2, 2, 2, dtype=torch.float64, device=device), "++--", 1, (4,))
    u, v = make(), make()
    if device != "cpu":
        P.einsum(SUB, u, v)                       # (the right shape has been planned)
    x = (u, v)[operand]
    for extents in ((1, 1, 1), (4, 4, 2)):
        x.data = torch.zeros(*extents, 2, 2, 2, 2, dtype=torch.float64, device=device)
        for _ in range(2):
            with pytest.raises(ValueError, match="reduced form must have shape"):
                P.einsum(SUB, u, v)


def test_gradients_are_planned_for_the_tensors_they_get(monkeypatch):
    runs = []
    monkeypatch.setattr(S, "_check_dense", lambda t: None)
    monkeypatch.setattr(S._Planned, "run", lambda self, *data, **kw: runs.append(
        [(d.c.dtype, tuple(d._dims)) == (S._DTYPE_CODE[t.dtype], tuple(t.shape[3:]))
         for d, t in zip((self.du, self.dv, self.dw), data)]))
    make = lambda: P.SymTensor(torch.zeros(2, 2, 2, 2, 3, 2, 3, dtype=torch.float64), "++--", 1, (2,))
    u, v = make(), make()
    call = S._Einsum(SUB, u, v, "f64")
    gw = torch.zeros(call.shape, dtype=torch.float64)
    for dtype in (torch.float64, torch.float32, torch.float64):
        for operand, (x, like) in enumerate(((v.data, u.data), (u.data, v.data))):
            call.gradient(operand, gw.to(dtype), x.to(dtype), torch.empty_like(like, dtype=dtype))
    assert len(runs) == 6 and all(all(r) for r in runs), runs
    with pytest.raises(ValueError, match="reduced form must have shape"):
        call.gradient(0, gw, v.data[:1], torch.empty_like(u.data))


@pytest.mark.gpu
def test_saved_tensor_hooks_may_change_the_storage_type():
    g = torch.Generator().manual_seed(7)
    make = lambda: P.SymTensor(torch.randn(3, 3, 3, 4, 5, 4, 5, dtype=torch.float64, generator=g).to("cuda:0"), "++--", 1, (3,))
    u, v = make(), make()

    def grads():
        a = P.SymTensor(u.data.detach().clone().requires_grad_(), u.signs, u.charge, u.group)
        b = P.SymTensor(v.data.detach().clone().requires_grad_(), v.signs, v.charge, v.group)
        w = P.einsum(SUB, a, b)
        (w.data * w.data.detach()).sum().backward()
        return a.data.grad, b.data.grad
    for hooks in (False, True, False):
        if hooks:
            with torch.autograd.graph.saved_tensors_hooks(lambda t: t.float(), lambda t: t):
                got = grads()
        else:
            want = got = grads()
        for x, y in zip(got, want):
            # (operands and gradients rounded to binary32; the products sum 60 binary64 terms)
            assert (x - y).abs().max() <= 8 * 2.0 ** -24 * y.abs().max() * 60
