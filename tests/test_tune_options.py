"""The tuner times one option of every launch (CPU)."""
import pytest

from paper_1111_1129_amd import _native as N
from paper_1111_1129_amd import lattice as L
from paper_1111_1129_amd.tune import SWEEPS, launch_options

CHUNKS = (1, 4, 16, 64, 0)


def launch(n, storage, kind, nt, chunk):
    code_bytes = 1 if kind.endswith("c8") else 2 if kind.endswith("c16") else 4
    st, out = N.lbm_sweep_launch(L.params(storage=storage, nontemporal=nt, xcd_chunk=chunk), n, 18,
                                 code_bytes, kind.startswith("inplace"))
    assert st == 0
    return out


@pytest.mark.parametrize("kind", SWEEPS)
@pytest.mark.parametrize("storage", ["f64", "f64s", "f32", "f32s", "f16s", "f16s12"])
@pytest.mark.parametrize("n", [17263, 1_000_000, 3_000_000, 5_000_000, 107_371_203])
def test_one_option_of_every_launch(n, storage, kind):
    kept = launch_options(n, storage, kind, CHUNKS)
    of = {launch(n, storage, kind, *o): o for o in kept}
    assert len(of) == len(kept)
    assert set(of) == {launch(n, storage, kind, nt, c) for nt in (False, True) for c in CHUNKS}
    for (_, stores, _), (nt, _) in of.items():
        assert nt == (stores == 2)
    if n == 17263:
        assert kept == [(False, 0)]
    if n == 107_371_203:
        assert len(kept) == (5 if kind.endswith("c8") or storage.startswith("f64") else 10)
