"""A forward run takes the codes of its own list only (CPU: refused before
anything is launched)."""
import pytest
import torch

from paper_1111_1129_amd import adjoint as AD
from paper_1111_1129_amd import lattice as L


def arrays(n, stride):
    codes = torch.zeros((18, stride), dtype=torch.int16)
    records = torch.zeros(((n + 255) // 256, 20), dtype=torch.int32)
    return L.Compressed(codes, records, n, 0, codes8=torch.zeros((18, stride), dtype=torch.int8))


@pytest.mark.parametrize("n,stride", [(299, 320), (301, 320), (300, 319), (40, 64)])
def test_codes_of_another_list_are_refused(n, stride):
    lat = L.Lattice((10, 10, 3), 0, "lex", 0, 300, 0, 320, None, None,
                    torch.zeros((18, 320), dtype=torch.int32))
    prm = L.params(storage="f64s")
    with pytest.raises(AssertionError):
        AD.forward_states(lat, prm, None, 2, 1, arrays(n, stride))
