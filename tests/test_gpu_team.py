"""Workgroups that share a system's sweeps: bitwise what one workgroup does, at
the edges of the multi-workgroup engine's layouts."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2506_21290_amd import flipmc  # noqa: E402

pytestmark = pytest.mark.gpu


def chain(M, T, k, nc, seed, fp32, sweeps, workgroups, **more):
    rng = np.random.default_rng(seed)
    n = int(np.ceil(M ** (1 / 3)))
    side = (3.0 * M / more.get("density", 1.2)) ** (1 / 3)
    at = np.sort(rng.permutation(n ** 3)[:M])
    com = (np.stack([at % n, (at // n) % n, at // (n * n)], axis=1) + 0.5) * (side / n)
    q = rng.normal(size=(M, 4))
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    types = np.argsort(rng.random((M, 3)), axis=1).astype(np.uint8)
    p = flipmc.mc_params_default(n_molecules=M, temperature=T, colours_per_axis=k, cells_per_side=nc, seed=seed,
                                 precision=flipmc.MC_FP32_DE if fp32 else flipmc.MC_FP64, workgroups=workgroups,
                                 gofr_interval=0, resum_interval=2, **more)
    s = flipmc.System(p, com=com, quat=q, types=types)
    s.decision_log(sweeps)
    s.sweep(sweeps)
    out = s.read_log(), s.get_state(), s.observables()
    s.close()
    return out


@pytest.mark.parametrize("M,k,nc,flags,want", [
    (64, 2, 2, 0, (flipmc.MC_ENGINE_SPREAD, 1)),      # one cell per colour
    (1000, 2, 4, 0, (flipmc.MC_ENGINE_SPREAD, 8)),    # fits one workgroup's LDS, faster on a workgroup per cell
    (1000, 2, 4, flipmc.MC_FLAG_SINGLE_WORKGROUP, (flipmc.MC_ENGINE_LDS, 1)),
    (2197, 2, 6, 0, (flipmc.MC_ENGINE_SPREAD, 27)),
    (2197, 2, 6, flipmc.MC_FLAG_SINGLE_WORKGROUP, (flipmc.MC_ENGINE_HBM, 1)),
])
def test_engine_names_what_a_sweep_launches(M, k, nc, flags, want):
    p = flipmc.mc_params_default(n_molecules=M, colours_per_axis=k, cells_per_side=nc, flags=flags)
    assert flipmc.mc_engine(p) == want


def test_long_runs_take_several_launches():
    # the workgroups that share a system are chosen at a launch, which is
    # therefore bounded; the chain goes on as in one launch
    p = flipmc.mc_params_default(n_molecules=343, temperature=1.5, colours_per_axis=2, cells_per_side=4, workgroups=8,
                                 precision=flipmc.MC_FP32_DE, resum_interval=0, gofr_interval=0)
    a, b = flipmc.System(p), flipmc.System(p)
    a.sweep(2000)
    b.sweep(2000)
    a.timing_enable(True)
    a.sweep(2990)  # no event before sweep 5000
    assert a.timing_read()["sweep_launches"] == 3
    for _ in range(13):
        b.sweep(230)
    sa, sb = a.get_state(), b.get_state()
    for f in ("com", "quat", "types", "e_acc", "sweep"):
        assert np.array_equal(sa[f], sb[f]), f


@pytest.mark.parametrize("M,k,nc,cells", [(1000, 2, 4, 8), (2197, 2, 6, 27)])
def test_workgroups_is_a_limit(M, k, nc, cells):
    for n in (2, 3, cells - 1, cells, cells + 1):
        p = flipmc.mc_params_default(n_molecules=M, colours_per_axis=k, cells_per_side=nc, workgroups=n)
        assert flipmc.mc_engine(p) == (flipmc.MC_ENGINE_SPREAD, min(n, cells))


@pytest.mark.parametrize("M,k,nc,workgroups", [
    (64, 2, 2, 0),       # one cell per colour: one workgroup's waves share it
    (83, 2, 2, 0),       # no whole groups of eight molecules
    (1000, 2, 2, 0),     # 125 molecules a cell, neighbourhoods too large to stage
    (217, 3, 6, 0),      # 27 colours of 8 cells
    (1001, 2, 4, 0),     # 8 workgroups, each ranking all molecules
    (2048, 2, 6, 0),     # the largest that each ranks alone
    (2049, 2, 6, 0),     # the smallest whose ranks are shared out
    (1000, 2, 4, 3),     # fewer workgroups than the 8 cells of a colour
    (2197, 2, 6, 3),     # fewer workgroups than cells of a colour: a cell per wave
    (8000, 2, 10, 4),    # the same with several cells a wave
    (2747, 2, 8, 0),     # 64 workgroups: barriers in groups
    (6001, 3, 18, 0),    # 216 workgroups, 125 cells in the stencil
])
@pytest.mark.parametrize("fp32", [False, True])
def test_team_equals_one_workgroup(M, k, nc, workgroups, fp32):
    n = 4
    l0, s0, o0 = chain(M, 1.1, k, nc, 7, fp32, n, 1)
    l1, s1, o1 = chain(M, 1.1, k, nc, 7, fp32, n, workgroups)
    for f in ("delta_e", "scale", "accepted", "exited", "move", "pair_terms"):
        assert np.array_equal(l0[f], l1[f]), f
    for f in ("com", "quat", "types", "e_acc", "sweep"):
        assert np.array_equal(s0[f], s1[f]), f
    for f in ("attempts", "accepts", "exits", "pair_terms", "pair_tests", "near_overflows"):
        assert np.array_equal(o0[f], o1[f]), f
    assert np.sum(o1["accepts"]) > 0 and (nc > 2 or M < 1000 or o1["near_overflows"] > 0)


@pytest.mark.parametrize("M,k,nc,density", [
    (60, 2, 2, 1.2),     # less than one entry a lane
    (500, 2, 4, 0.6),    # one to two
    (1000, 2, 4, 1.2),   # up to three
    (1000, 2, 4, 2.0),   # the last of the list beyond three a lane
])
@pytest.mark.parametrize("fp32", [False, True])
def test_near_entries_of_either_state(M, k, nc, density, fp32):
    # in LDS a lane holds its near entries, FP64 in HBM reads them at each trial
    one = flipmc.MC_FLAG_SINGLE_WORKGROUP
    l0, s0, o0 = chain(M, 3.0, k, nc, 11, fp32, 3, 1, density=density, flags=one)
    l1, s1, o1 = chain(M, 3.0, k, nc, 11, fp32, 3, 1, density=density, flags=one | flipmc.MC_FLAG_HBM_STATE)
    for f in ("delta_e", "scale", "accepted", "exited", "move", "pair_terms"):
        assert np.array_equal(l0[f], l1[f]), f
    for f in ("com", "quat", "types", "e_acc", "sweep"):
        assert np.array_equal(s0[f], s1[f]), f
    for f in ("attempts", "accepts", "exits", "pair_terms", "pair_tests", "near_overflows"):
        assert np.array_equal(o0[f], o1[f]), f
    assert np.sum(o1["accepts"]) > 0


@pytest.mark.parametrize("fp32", [False, True])
def test_cells_whose_first_trials_all_exit(fp32):
    # 125 molecules a cell and steps longer than it: 0.94 of the trials leave
    # their cell, so in some 2 % of the cells the first 64 all do, and the next
    # 61 follow with no trial evaluated in between
    step = dict(p_flip=0.0, p_translate=1.0, max_displacement=8.9)
    l0, s0, o0 = chain(27000, 1.1, 2, 6, 3, fp32, 2, 1, **step)
    l1, s1, o1 = chain(27000, 1.1, 2, 6, 3, fp32, 2, 0, **step)
    assert np.mean(l0["exited"]) > 0.9
    for f in ("delta_e", "accepted", "exited", "pair_terms"):
        assert np.array_equal(l0[f], l1[f]), f
    for f in ("com", "quat", "types", "e_acc"):
        assert np.array_equal(s0[f], s1[f]), f
    for f in ("attempts", "accepts", "exits"):
        assert np.array_equal(o0[f], o1[f]), f


@pytest.mark.parametrize("M,nc,workgroups,fp32,more", [
    (40000, 18, 0, True, {}),        # more cells of a colour than workgroups: a cell per wave
    (40000, 18, 0, False, {}),
    (40000, 18, 3, True, {}),        # several cells a wave
    (40000, 12, 0, True, {}),        # 216 cells of a colour: a cell per workgroup
    (9000, 34, 0, True, dict(density=0.05)),  # it is the cells that are too many, most of them empty
])
def test_lists_beyond_lds(M, nc, workgroups, fp32, more):
    # the cell lists do not fit a workgroup's LDS, and the workgroups build them
    # together in the system's buffer
    l0, s0, _ = chain(M, 1.1, 2, nc, 5, fp32, 2, 1, **more)
    l1, s1, _ = chain(M, 1.1, 2, nc, 5, fp32, 2, workgroups, **more)
    assert np.array_equal(l0["delta_e"], l1["delta_e"]) and np.array_equal(l0["accepted"], l1["accepted"])
    for f in ("com", "quat", "types", "e_acc"):
        assert np.array_equal(s0[f], s1[f]), f


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("limit", [12, 0])
def test_batch_of_short_and_long_systems(fp32, limit):
    # a run of all remaining sweeps puts short systems one after another on one
    # workgroup and gives the long ones several (a cell per workgroup or per
    # wave); each ends as it does alone
    sizes = [(64, 2, 2)] * 9 + [(1000, 2, 4), (1728, 2, 6), (2197, 2, 6)]

    def system(i, M, k, nc, **kw):
        p = flipmc.mc_params_default(n_molecules=M, temperature=1.3, colours_per_axis=k, cells_per_side=nc, seed=i,
                                     precision=flipmc.MC_FP32_DE if fp32 else flipmc.MC_FP64, resum_interval=7,
                                     gofr_interval=5, workgroups=0)
        return flipmc.System(p, **kw)

    alone = []
    for i, (M, k, nc) in enumerate(sizes):
        s = system(i, M, k, nc)
        s.sweep(21)
        alone.append((s.get_state(), s.observables()))
        s.close()
    b = flipmc.Batch(len(sizes), flipmc.MC_FP32_DE if fp32 else flipmc.MC_FP64)
    b.set_workgroups(limit)
    systems = [system(i, M, k, nc, stream=b.stream) for i, (M, k, nc) in enumerate(sizes)]
    for s in systems:
        b.add(s, 21)
    left = len(systems)
    for _ in range(100):
        b.run(0)
        left -= len(b.poll())
        if not left:
            break
    assert left == 0
    for s, (ref, obs) in zip(systems, alone):
        st, o = s.get_state(), s.observables()
        for f in ("com", "quat", "types", "e_acc", "sweep"):
            assert np.array_equal(st[f], ref[f]), f
        for f in ("accepts", "pair_terms", "gofr_all", "c2", "e_resum"):
            assert np.array_equal(o[f], obs[f]), f
    b.close()


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("limit", [24, 40, 0])
def test_batch_too_wide_for_its_least_work(fp32, limit):
    # each of these systems takes the least work on several workgroups, and all
    # of them more than the limit: some keep fewer, and each ends as it does alone
    sizes = [(2197, 2, 6), (1728, 2, 6), (1000, 2, 4)] * 8

    def system(i, M, k, nc, **kw):
        p = flipmc.mc_params_default(n_molecules=M, temperature=1.3, colours_per_axis=k, cells_per_side=nc, seed=i % 3,
                                     precision=flipmc.MC_FP32_DE if fp32 else flipmc.MC_FP64, gofr_interval=0)
        return flipmc.System(p, **kw)

    alone = []
    for i, (M, k, nc) in enumerate(sizes[:3]):
        s = system(i, M, k, nc)
        s.sweep(6)
        alone.append(s.get_state())
        s.close()
    b = flipmc.Batch(len(sizes), flipmc.MC_FP32_DE if fp32 else flipmc.MC_FP64)
    b.set_workgroups(limit)
    systems = [system(i, M, k, nc, stream=b.stream) for i, (M, k, nc) in enumerate(sizes)]
    for s in systems:
        b.add(s, 6)
    left = len(systems)
    for _ in range(100):
        b.run(0)
        left -= len(b.poll())
        if not left:
            break
    assert left == 0
    for i, s in enumerate(systems):
        st = s.get_state()
        for f in ("com", "quat", "types", "e_acc", "sweep"):
            assert np.array_equal(st[f], alone[i % 3][f]), f
    b.close()


@pytest.mark.parametrize("count", [40, 129])
def test_frames_of_many_systems(count):
    # up to 128 systems take their g(r) frames on many workgroups each, more on
    # one: the same counts as alone
    def system(i, **kw):
        p = flipmc.mc_params_default(n_molecules=343, temperature=1.3, colours_per_axis=2, cells_per_side=4, seed=i % 3,
                                     precision=flipmc.MC_FP32_DE, gofr_interval=3, resum_interval=0)
        return flipmc.System(p, **kw)

    alone = []
    for i in range(3):
        s = system(i)
        s.sweep(7)
        alone.append(s.observables())
        s.close()
    b = flipmc.Batch(count, flipmc.MC_FP32_DE)
    systems = [system(i, stream=b.stream) for i in range(count)]
    for s in systems:
        b.add(s, 7)
    left = count
    for _ in range(20):
        b.run(0)
        left -= len(b.poll())
        if not left:
            break
    assert left == 0
    for i, s in enumerate(systems):
        o = s.observables()
        assert o["n_gofr_frames"] == 2
        for f in ("gofr_all", "gofr_inter", "e_acc", "accepts"):
            assert np.array_equal(o[f], alone[i % 3][f]), f
    b.close()


def test_time_slices_of_every_engine_run_beside_each_other():
    # a time slice has at most three launches, one per stream: with systems on
    # one HBM workgroup, those with several workgroups take one way, and each
    # ends as it does alone
    sizes = [(8000, 2, 10, 60), (125, 2, 2, 400), (125, 2, 2, 300), (343, 2, 4, 200)] + [(2197, 2, 6, 40)] * 4

    def system(i, M, k, nc, **kw):
        p = flipmc.mc_params_default(n_molecules=M, temperature=1.3, colours_per_axis=k, cells_per_side=nc, seed=i,
                                     precision=flipmc.MC_FP32_DE, resum_interval=0, gofr_interval=0)
        return flipmc.System(p, **kw)

    b = flipmc.Batch(len(sizes), flipmc.MC_FP32_DE)
    b.set_workgroups(16)
    systems = [system(i, M, k, nc, stream=b.stream) for i, (M, k, nc, _) in enumerate(sizes)]
    for s, (_, _, _, n) in zip(systems, sizes):
        b.add(s, n)
    launched, left = [], len(systems)
    for _ in range(500):
        launched.append(b.run(10000))
        left -= len(b.poll())
        if not left:
            break
    assert left == 0 and max(launched) == 3
    for i, (s, (M, k, nc, n)) in enumerate(zip(systems, sizes)):
        alone = system(i, M, k, nc)
        alone.sweep(n)
        st, ref = s.get_state(), alone.get_state()
        for f in ("com", "quat", "types", "e_acc", "sweep"):
            assert np.array_equal(st[f], ref[f]), f
    b.close()


def test_time_slices_of_more_systems_than_compute_units_are_fair():
    # small systems in LDS and as many large ones, some of which take the
    # multi-workgroup engine on one workgroup: each gets about the same time,
    # in sweeps of it alone on one workgroup (the engines differ by 1.5 there and
    # the cost model by 1.3 either way, so a third counts as the same; where the
    # launch that started first kept the device it was a tenth)
    kinds = [(343, 2, 4), (2744, 2, 8)]
    cus = torch.cuda.get_device_properties(0).multi_processor_count

    def params(kind, seed):
        M, k, nc = kinds[kind]
        return flipmc.mc_params_default(n_molecules=M, temperature=1.5, colours_per_axis=k, cells_per_side=nc, seed=seed,
                                        precision=flipmc.MC_FP32_DE, resum_interval=0, obs_interval=0,
                                        gofr_interval=0, workgroups=1)

    alone = []
    for kind in (0, 1):
        s = flipmc.System(params(kind, 1))
        s.sweep(20)
        s.energy()
        t0 = time.perf_counter()
        s.sweep(50)
        s.energy()
        alone.append((time.perf_counter() - t0) / 50)
        s.close()
    b = flipmc.Batch(2 * cus, flipmc.MC_FP32_DE)
    systems = []
    for i in range(2 * cus):
        p = params(i % 2, i + 1)
        p.workgroups = 0
        systems.append(flipmc.System(p, stream=b.stream))
        b.add(systems[-1], 10**6)
    for _ in range(24):
        b.run(100000)
        b.poll()
    done = [np.mean([s.get_state()["sweep"] for s in systems[kind::2]]) * alone[kind] for kind in (0, 1)]
    assert 1 / 3 < done[0] / done[1] < 3, (done, alone)
    b.close()


@pytest.mark.parametrize("same", [True, False])
def test_two_batches_in_turn(same):
    # batches on one stream share their side streams; batches on two do not
    sizes = [(64, 2, 2), (216, 3, 6), (1000, 2, 4), (1728, 2, 6)]

    def systems(stream=None):
        return [flipmc.System(flipmc.mc_params_default(n_molecules=M, temperature=1.3, colours_per_axis=k,
                                                       cells_per_side=nc, seed=i, resum_interval=7,
                                                       precision=flipmc.MC_FP32_DE), stream=stream)
                for i, (M, k, nc) in enumerate(sizes)]

    alone = systems()
    for s in alone:
        s.sweep(12)
    two = [flipmc.Batch(8, flipmc.MC_FP32_DE), flipmc.Batch(8, flipmc.MC_FP32_DE,
                                                            stream=None if same else torch.cuda.Stream())]
    assert (two[0].aux_stream == two[1].aux_stream) is same
    assert len({b.aux_stream for b in two} | {b.hbm_stream for b in two}) == (2 if same else 4)
    torch.cuda.synchronize()
    sets = [systems(b.stream) for b in two]
    for b, own in zip(two, sets):
        for s in own:
            b.add(s, 12)
    left = [len(sizes)] * 2
    for _ in range(50):
        for x, b in enumerate(two):
            b.run(0)
        for x, b in enumerate(two):
            left[x] -= len(b.poll())
        if left == [0, 0]:
            break
    assert left == [0, 0]
    for own in sets:
        for s, ref in zip(own, alone):
            st, r = s.get_state(), ref.get_state()
            for f in ("com", "quat", "types", "e_acc", "sweep"):
                assert np.array_equal(st[f], r[f]), f
    for b in two:
        b.close()
