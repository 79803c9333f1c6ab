"""The flexible sweep kernel's rows of lanes at their edges: neighbour lists
that fit, that do not fit (their rows walk the 27 cells) and both in one
system, and a system whose atoms 16 bits cannot index (no lists at all)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import test_gpu_flex as flexgpu  # noqa: E402
from paper_2506_21290_amd import flipmc  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("body,density", [("triangle", 2.7), ("triangle", 3.4), ("square", 1.2), ("tetrahedron", 2.7)])
def test_lists_that_overflow_match_the_oracle(monkeypatch, body, density):
    # about 16.5 density atoms lie within r_c + 2 sqrt(3) d of an atom: 20 at
    # density 1.2, 45 (some lists overflow) and 56 (most do)
    geometry = {"triangle": flipmc.MC_TRIANGLE, "square": flipmc.MC_SQUARE, "tetrahedron": flipmc.MC_TETRAHEDRON}
    monkeypatch.setitem(flexgpu.CASES, "dense", (geometry[body], 343, 2.0, 3, 3, density))
    s, o, resyncs = flexgpu.run("dense", 2)
    assert resyncs == 0
    e, _, drift = s.energy()
    assert abs(drift) <= 1e-11 * abs(e)


def test_system_beyond_16_bit_atom_indices():
    p = flipmc.mcf_params_default(flipmc.MC_TRIANGLE, n_molecules=28 ** 3, temperature=2.0, gofr_interval=0)
    s = flipmc.FlexSystem(p)
    e0 = s.energy()[0]
    s.sweep(1)
    e, _, drift = s.energy()
    o = s.observables()
    st = s.get_state()
    assert o["attempts"].sum() == st["types"].size == 65856
    assert e < e0  # the lattice start's overlaps relax
    assert abs(drift) <= 1e-11 * abs(e0)
    assert np.all((st["pos"] >= 0.0) & (st["pos"] < flipmc.mcf_geometry(p)[0]))
