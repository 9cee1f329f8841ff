"""What einsum refuses: operands whose data no longer has the reduced form's shape."""
import pytest
import torch

import paper_2007_08056_amd as P

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
