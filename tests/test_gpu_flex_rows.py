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


@pytest.mark.parametrize("k,nc", [(3, 3), (3, 6)])
def test_lists_in_a_dilute_box(k, nc):
    # neighbours are selected in FP32: a drop in a box of side 1e8, where a float
    # holds a coordinate of a cell to 1 or more, keeps every pair all the same
    M, side = 125, 1e8
    rng = np.random.default_rng(9)
    c = np.stack(np.meshgrid(*[np.arange(5)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    b = 0.9608971989592554
    shape = np.array([[b / np.sqrt(3), 0, 0], [-b / np.sqrt(12), b / 2, 0], [-b / np.sqrt(12), -b / 2, 0]])
    q = np.linalg.qr(rng.normal(size=(M, 3, 3)))[0]
    pos = 0.93 * side + 1.5 * c[:, None, :] + np.einsum("mij,sj->msi", q, shape)
    types = np.argsort(rng.random((M, 3)), axis=1).astype(np.uint8)
    p = flipmc.mcf_params_default(flipmc.MC_TRIANGLE, n_molecules=M, temperature=1.0, seed=3, resum_interval=0,
                                  density=3.0 * M / side ** 3, colours_per_axis=k, cells_per_side=nc)
    s = flipmc.FlexSystem(p, pos=pos, types=types)
    s.decision_log(5)
    s.sweep(5)
    log = s.read_log()
    assert log["accepted"].sum() > 100 and log["pair_terms"].sum() > 10 * len(log)
    # differences of coordinates are exact and displacements those of the stored
    # coordinates, so E_acc is off by the rounding of some 30 terms a move only
    scale = log["scale"][log["accepted"] == 1].sum()
    _, _, drift = s.energy()
    assert abs(drift) <= 32 * 2.2e-16 * scale
    s.close()


@pytest.mark.parametrize("body", [flipmc.MC_TRIANGLE, flipmc.MC_SQUARE, flipmc.MC_TETRAHEDRON])
def test_large_moves_of_an_overlapping_start_add_up(body):
    # moves that change the energy by more than 1e4 enter E_acc by the sum over
    # the stencil instead of the one over the rows: the same energy to rounding
    n = 3 if body == flipmc.MC_TRIANGLE else 4
    M = 131
    rng = np.random.default_rng(5)
    side = (n * M / 1.2) ** (1 / 3)
    c = int(np.ceil(M ** (1 / 3)))
    at = np.sort(rng.permutation(c ** 3)[:M])
    com = (np.stack([at % c, (at // c) % c, at // (c * c)], axis=1) + 0.5) * (side / c)
    b = 0.9608971989592554
    shape = {3: np.array([[b / np.sqrt(3), 0, 0], [-b / np.sqrt(12), b / 2, 0], [-b / np.sqrt(12), -b / 2, 0]]),
             4: np.array([[b / 2, b / 2, 0], [-b / 2, b / 2, 0], [-b / 2, -b / 2, 0], [b / 2, -b / 2, 0]])}[n]
    if body == flipmc.MC_TETRAHEDRON:
        shape = b / np.sqrt(8) * np.array([[1, 1, 1], [1, -1, -1], [-1, 1, -1], [-1, -1, 1]])
    q = np.linalg.qr(rng.normal(size=(M, 3, 3)))[0]
    pos = com[:, None, :] + np.einsum("mij,sj->msi", q, shape)
    types = np.argsort(rng.random((M, n)), axis=1).astype(np.uint8)
    s = flipmc.FlexSystem(flipmc.mcf_params_default(body, n_molecules=M, temperature=1.0, seed=3, resum_interval=0),
                          pos=pos, types=types)
    e0 = s.get_state()["e_acc"]
    s.decision_log(2)
    s.sweep(2)
    log, e = s.read_log(), s.get_state()["e_acc"]
    de = log["delta_e"][log["accepted"] == 1]
    assert np.abs(de).max() > 1e4
    # each sum rounds some 40 terms of up to |dE|, and E_acc adds them one by one
    assert abs(e - (e0 + de.sum())) <= 1e-13 * (abs(e0) + np.abs(de).sum())
    s.close()
