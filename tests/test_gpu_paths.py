"""Kernel paths at the sizes and positions where they can go wrong, against
the FP64 oracle (bars as in test_gpu_parity.py: FP64 scenes to 1e-9, FP32
within 1e-4 of the displacement and 1e-3 of the stress)."""
import numpy as np
import pytest

import oracle
from paper_1909_13380_amd import scenes

pytestmark = pytest.mark.gpu

BARS = {"fp64": (1e-9, 1e-9), "fp32": (1e-4, 1e-3)}


@pytest.fixture(scope="module")
def mp():
    from paper_1909_13380_amd import mpmx
    return mpmx


@pytest.fixture(scope="module")
def ctx(mp):
    c = mp.Context(0)
    yield c
    c.close()


def rel(a, b):
    nb = np.linalg.norm(b)
    return np.linalg.norm(np.asarray(a) - np.asarray(b)) / (nb if nb > 0 else 1.0)


def check(name, got, ref, x0, bars):
    eu, es = rel(got["x"] - x0, ref["x"] - x0), rel(got["stress"], ref["stress"])
    print(f"[{name}] err_u={eu:.3e} err_sigma={es:.3e}", flush=True)
    assert eu <= bars[0] and es <= bars[1], (name, eu, es)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("algo", [scenes.USF, scenes.USL, scenes.MUSL])
def test_gimp_supports_at_their_joins(ctx, mp, algo, prec):
    """Particles at the cell coordinates where a GIMP support changes its
    first node (1/4), its weights change piece (3/4, also the cell's faces
    and centre), and a hair on either side of each."""
    sc = scenes.random_block(n_cells=(6, 5, 4), shape=1, seed=61, vel=0.5, stress_scale=2e3,
                             material=scenes.drucker_prager(psi_deg=5, c=1e3))
    sc["scheme"]["algo"] = algo
    h = sc["mesh"]["h"]
    rng = np.random.default_rng(61)
    joins = np.array([0.0, 1e-13, 0.25 - 1e-13, 0.25, 0.25 + 1e-13, 0.5, 0.75 - 1e-13, 0.75, 0.75 + 1e-13, 1 - 1e-13])
    cell = np.floor(sc["x"] / h)
    frac = rng.choice(joins, size=sc["x"].shape)
    frac[(cell == 0) & (frac < 0.2)] = 0.5          # a particle on the floor itself may leave the mesh
    sc["x"] = (cell + frac) * h
    s = ctx.create_scene(sc, precision=mp.FP64 if prec == "fp64" else mp.FP32)
    s.step(4)
    check(f"gimp-joins/{algo}/{prec}", s.read(), oracle.run(sc, 4), sc["x"], BARS[prec])
    s.destroy()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 511, 512, 513, 1500])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_read_returns_every_row_in_input_order(ctx, mp, prec, n):
    """Load and read at the edges of a wavefront and of the read's workgroup
    pass, before and after a reorder, all fields or some: the inputs come back
    row by row (values that FP32 holds, so exactly) and in place, and nothing
    past the last row is written."""
    import torch
    sc = scenes.random_block(n_cells=(6, 6, 6), mesh_cells=(12, 10, 9), seed=62, vel=0.3, stress_scale=2e3)
    pick = np.random.default_rng(n).permutation(len(sc["x"]))[:n]
    sc.update({k: np.ascontiguousarray(sc[k][pick]) for k in ("x", "v", "stress", "vol", "mass")})
    s = ctx.create_scene(sc, precision=mp.FP64 if prec == "fp64" else mp.FP32)
    want = {k: sc[k] for k in ("x", "v", "stress", "vol")}
    c = np.floor(sc["x"] / sc["mesh"]["h"]).astype(np.int64)
    want["cell"] = (c[:, 0] + 12 * (c[:, 1] + 10 * c[:, 2])).astype(np.int32)
    for k, a in s.read().items():
        np.testing.assert_array_equal(a, want[k], err_msg=k)
    s.step(1)
    host = s.read()
    check(f"read/{n}/{prec}", host, oracle.run(sc, 1), sc["x"], BARS[prec])
    for fields in (("x", "v", "stress", "vol", "cell"), ("stress",), ("cell", "x")):
        pad = {k: torch.full((np.asarray(host[k]).size + 8,), -7, dtype=torch.int32 if k == "cell" else torch.float64,
                             device="cuda") for k in fields}
        torch.cuda.synchronize()
        s.read(device_out=pad)
        for k in fields:
            got = pad[k].cpu().numpy()
            np.testing.assert_array_equal(got[:-8], np.asarray(host[k]).reshape(-1), err_msg=k)
            assert (got[-8:] == -7).all(), k
    s.destroy()


@pytest.mark.parametrize("noalloc", [False, True])
def test_known_reorders_run_phase_by_phase(ctx, mp, noalloc):
    """Scenes whose reorder the host knows of (fresh, or always sorting) in
    batches with ones it does not know of, an empty one and one asked for no
    steps, over three calls: each equals the oracle, and each always-sorting
    scene counts a reorder per step."""
    cells = [(9, 7, 6), (3, 3, 2), (5, 6, 4), (2, 2, 2), (4, 3, 3)]
    scs = [scenes.random_block(n_cells=c, mesh_cells=tuple(3 * k + 5 for k in c), seed=70 + i, vel=1.0, stress_scale=1e3)
           for i, c in enumerate(cells)]
    for k in ("x", "v", "stress", "vol", "mass"):
        scs[3][k] = scs[3][k][:0]
    always = [False, True, False, False, True]
    ss = [ctx.create_scene(sc, precision=mp.FP64, sort_policy=mp.SORT_ALWAYS if a else mp.SORT_ON_DEMAND)
          for sc, a in zip(scs, always)]
    steps = [[3, 2, 0, 2, 0], [0, 4, 5, 3, 0], [6, 3, 2, 1, 4]]
    for call in steps:
        (ctx.batch_step_noalloc if noalloc else ctx.batch_step)(ss, call)
    for i, (sc, s, a) in enumerate(zip(scs, ss, always)):
        k = sum(call[i] for call in steps)
        st = s.stats()
        assert st["error_bits"] == 0 and st["steps_done"] == k, (i, st)
        if a:
            assert st["n_sorts"] == k, (i, st)
        if len(sc["x"]):
            check(f"known-reorders/{i}/{noalloc}", s.read(), oracle.run(sc, k), sc["x"], BARS["fp64"])
        s.destroy()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("algo", [scenes.USF, scenes.USL, scenes.MUSL])
def test_isoparametric_location_of_fast_particles(ctx, mp, algo, prec):
    """A body that crosses most of a cell per step on strongly distorted
    cells: the location of a moved particle starts from the step matrix of
    its previous place, far from the new one, or walks into another cell."""
    base = scenes.random_block(n_cells=(6, 6, 5), mesh_cells=(16, 12, 10), h=0.05, seed=63, vel=2.0, dt=1e-4,
                               material=scenes.drucker_prager(psi_deg=5, c=1e3), stress_scale=2e3,
                               bc=scenes.walls(floor=scenes.FREE, sides=scenes.FREE))
    base["x"] = base["x"] + np.array([0.0, 0.0, 0.1])
    base["v"] = base["v"] + np.array([400.0, -150.0, 90.0])
    base["scheme"]["algo"] = algo
    sc = scenes.distort(base, amp=0.35, seed=64)
    s = ctx.create_scene(sc, precision=mp.FP64 if prec == "fp64" else mp.FP32)
    s.step(3)
    check(f"iso-fast/{algo}/{prec}", s.read(), oracle.run(sc, 3), sc["x"], BARS[prec])
    s.destroy()


def _flying(seed, v, n_cells=(9, 7, 6), shape=0, vel=2.0):
    sc = scenes.random_block(n_cells=n_cells, mesh_cells=(24, 20, 14), seed=seed, vel=vel, dt=1e-4, stress_scale=2e3,
                             shape=shape, material=scenes.drucker_prager(psi_deg=5, c=1e3),
                             bc=scenes.walls(floor=scenes.FREE, sides=scenes.FREE))
    sc["x"] = sc["x"] + np.array([-0.1, 0.05, 0.1])
    sc["v"] = sc["v"] + np.asarray(v, dtype=np.float64)
    return sc


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["linear", "gimp", "iso", "pic"])
def test_steps_in_one_launch_on_uneven_batches(ctx, mp, kind, prec):
    """Batches small enough for all their steps to run in one launch: scenes of
    1 to 14 items that end after different steps (none, one, ...), some fast
    enough to reorder several times on the way, over three calls."""
    shape = 1 if kind == "gimp" else 0
    big = [(5, 4, 3), (6, 5, 3)] if kind == "iso" else [(9, 7, 6), (12, 8, 7)]   # the oracle's location is slow
    scs = [_flying(80, (150.0, -60.0, 40.0), big[0], shape), _flying(81, (0.0, 0.0, 0.0), (4, 3, 3), shape),
           _flying(82, (-30.0, 10.0, 90.0), big[1], shape), _flying(83, (5.0, 0.0, 0.0), (1, 1, 1), shape)]
    if kind == "pic":
        for sc in scs:
            sc["scheme"]["velocity_update"] = scenes.PIC
    if kind == "iso":
        scs = [scenes.distort(sc, amp=0.2, seed=84) for sc in scs]
    ss = [ctx.create_scene(sc, precision=mp.FP64 if prec == "fp64" else mp.FP32) for sc in scs]
    calls = [[12, 3, 7, 1], [9, 0, 13, 2], [4, 17, 0, 20]]
    for call in calls:
        ctx.batch_step(ss, call)
    for i, (sc, s) in enumerate(zip(scs, ss)):
        k = sum(c[i] for c in calls)
        st = s.stats()
        assert st["error_bits"] == 0 and st["steps_done"] == k, (i, st)
        if i == 0:
            assert 2 <= st["n_sorts"] < k, st
        check(f"steps/{kind}/{prec}/{i}", s.read(), oracle.run(sc, k), sc["x"], BARS[prec])
        s.destroy()


def test_steps_in_one_launch_stop_at_an_error(ctx, mp):
    """A scene that leaves the mesh stops there, as the one-step calls stop
    it; the others of its batch go on."""
    scs = [_flying(85, (0.0, 0.0, 500.0)), _flying(86, (0.0, 0.0, 0.0)), _flying(87, (60.0, 0.0, 0.0))]
    one = ctx.create_scene(scs[0], precision=mp.FP64)
    for _ in range(40):
        one.step(1)
    want = one.stats()
    ss = [ctx.create_scene(sc, precision=mp.FP64) for sc in scs]
    ctx.batch_step(ss, [40, 40, 25])
    st = ss[0].stats()
    assert st["error_bits"] == want["error_bits"] == mp.ERRBIT_OUT_OF_MESH, (st, want)
    assert 0 < st["steps_done"] == want["steps_done"] < 40, (st, want)
    for i, k in ((1, 40), (2, 25)):
        assert ss[i].stats()["steps_done"] == k
        check(f"steps-error/{i}", ss[i].read(), oracle.run(scs[i], k), scs[i]["x"], BARS["fp64"])
    for s in [one] + ss:
        s.destroy()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_steps_in_one_launch_with_many_items_per_workgroup(ctx, mp, prec):
    """A sparse cloud that expands from 216 bricks to over 2500, so that a
    workgroup's items outgrow what it keeps of them from step to step."""
    sc = scenes.random_block(n_cells=(23, 23, 23), mesh_cells=(72, 72, 72), seed=5, vel=0.2, dt=1e-4,
                             gravity=(0.0, 0.0, 0.0), bc=scenes.walls(floor=scenes.FREE, sides=scenes.FREE),
                             material=scenes.elastic(E=1e3), jitter=0.3)
    pick = np.random.default_rng(5).permutation(len(sc["x"]))[::8]
    sc.update({k: np.ascontiguousarray(sc[k][pick]) for k in ("x", "v", "stress", "vol", "mass")})
    h = sc["mesh"]["h"]
    sc["x"] = sc["x"] + np.array([0.0, 0.0, 24 * h])
    sc["v"] = sc["v"] + 500.0 * (sc["x"] - 36 * h)
    s = ctx.create_scene(sc, precision=mp.FP64 if prec == "fp64" else mp.FP32)
    s.step(30)
    st = s.stats()
    assert st["error_bits"] == 0 and st["n_sorts"] >= 2 and st["n_items"] > 8 * 256, st
    check(f"steps-many-items/{prec}", s.read(), oracle.run(sc, 30), sc["x"], BARS[prec])
    s.destroy()


def test_steps_in_more_launches_than_one(ctx, mp):
    """More steps in a call than one launch takes (1024), at rest under
    gravity on a fixed floor."""
    sc = scenes.random_block(n_cells=(3, 2, 2), mesh_cells=(9, 8, 6), seed=88, vel=0.1)
    s = ctx.create_scene(sc, precision=mp.FP64)
    s.step(2100)
    assert s.stats()["steps_done"] == 2100
    check("steps-launches", s.read(), oracle.run(sc, 2100), sc["x"], BARS["fp64"])
    s.destroy()


def test_steps_in_one_launch_from_two_threads(mp):
    """Two contexts, each with a thread and a stream of its own, step batches
    that both ask for most of the device: neither waits for the other's
    workgroups to end, and both are right."""
    import threading
    sc = scenes.random_block(n_cells=(23, 22, 23), mesh_cells=(40, 40, 40), seed=89, vel=0.5, stress_scale=1e3)
    ref = oracle.run(sc, 60)
    out = [None, None]

    def work(i):
        c = mp.Context(0)
        s = c.create_scene(sc, precision=mp.FP64)
        for _ in range(3):
            s.step(20)
        out[i] = (s.read(), s.stats())
        s.destroy()
        c.close()

    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for i in range(2):
        got, st = out[i]
        assert st["error_bits"] == 0 and st["steps_done"] == 60, st
        check(f"steps-threads/{i}", got, ref, sc["x"], BARS["fp64"])


@pytest.mark.parametrize("n", [9300, 9361, 9362, 9363, 9707, 9708, 9709, 9800])
def test_host_arrays_around_the_pinned_memory_size(ctx, mp, n):
    """Scenes whose host arrays just fit, or do not fit, 1 MiB (112 bytes a
    particle on the way in, 108 on the way out): every value comes back, from
    two scenes in turn."""
    sc = scenes.random_block(n_cells=(11, 11, 11), mesh_cells=(22, 16, 14), seed=90, vel=0.3, stress_scale=2e3)
    rng = np.random.default_rng(n)
    scs = []
    for _ in range(2):
        pick = rng.permutation(len(sc["x"]))[:n]
        scs.append(dict(sc, **{k: np.ascontiguousarray(sc[k][pick]) for k in ("x", "v", "stress", "vol", "mass")}))
    ss = [ctx.create_scene(c, precision=mp.FP64) for c in scs]
    for c, s in zip(scs, ss):
        got = s.read()
        for k in ("x", "v", "stress", "vol"):
            np.testing.assert_array_equal(got[k], c[k], err_msg=k)
        s.destroy()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("algo", [scenes.USF, scenes.USL, scenes.MUSL])
def test_gimp_particles_alone_and_in_pairs(ctx, mp, algo, prec):
    """Cells of one to eight particles at random places: a thread's two
    particles share a cell or do not, through the separate kernels (the
    allocation-free call) and the default path."""
    sc = scenes.random_block(n_cells=(9, 6, 5), mesh_cells=(18, 13, 11), shape=1, seed=91, vel=0.5, stress_scale=2e3,
                             material=scenes.drucker_prager(psi_deg=5, c=1e3))
    sc["scheme"]["algo"] = algo
    h = sc["mesh"]["h"]
    rng = np.random.default_rng(91)
    keep = rng.random(len(sc["x"])) < 0.6
    sc.update({k: np.ascontiguousarray(sc[k][keep]) for k in ("x", "v", "stress", "vol", "mass")})
    sc["x"] = (np.floor(sc["x"] / h) + rng.uniform(0.02, 0.98, size=sc["x"].shape)) * h
    ref = oracle.run(sc, 4)
    for noalloc in (False, True):
        s = ctx.create_scene(sc, precision=mp.FP64 if prec == "fp64" else mp.FP32)
        (ctx.batch_step_noalloc if noalloc else ctx.batch_step)([s], [4])
        check(f"gimp-pairs/{algo}/{prec}/{noalloc}", s.read(), ref, sc["x"], BARS[prec])
        s.destroy()


def test_steps_in_one_launch_of_scenes_that_end_with_many_items_left(ctx, mp):
    """Clouds that spread to over 2400 bricks each in one batch, then a call in
    which they end after different steps: a workgroup reloads the items it
    keeps several times a stage, with finished scenes' items among them."""
    scs = []
    for seed in range(92, 98):
        sc = scenes.random_block(n_cells=(11, 11, 11), mesh_cells=(72, 72, 72), seed=seed, vel=0.2, dt=1e-4,
                                 gravity=(0.0, 0.0, 0.0), bc=scenes.walls(floor=scenes.FREE, sides=scenes.FREE),
                                 material=scenes.elastic(E=1e3), jitter=0.3)
        mid = 36 * sc["mesh"]["h"]
        sc["x"] = sc["x"] - 0.5 * (sc["x"].min(0) + sc["x"].max(0)) + mid
        sc["v"] = sc["v"] + 400.0 * (sc["x"] - mid)
        scs.append(sc)
    ss = [ctx.create_scene(sc, precision=mp.FP64) for sc in scs]
    calls = [[112] * 6, [3, 14, 1, 9, 6, 12]]
    for call in calls:
        ctx.batch_step(ss, call)
    for i, (sc, s) in enumerate(zip(scs, ss)):
        k = sum(c[i] for c in calls)
        st = s.stats()
        assert st["error_bits"] == 0 and st["steps_done"] == k and st["n_items"] > 2400, (i, st)
        check(f"steps-uneven-many/{i}", s.read(), oracle.run(sc, k), sc["x"], BARS["fp64"])
        s.destroy()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("mesh", [(40, 36, 24), (76, 72, 60), (100, 90, 80)])
def test_reorders_inside_a_launch_on_large_meshes(ctx, mp, mesh, prec):
    """Small fast bodies on meshes of 500 to 13000 bricks, stepped together:
    a few, some or many workgroups share each reorder."""
    scs = []
    for seed, v in ((101, (150.0, -50.0, 30.0)), (102, (-90.0, 60.0, 20.0))):
        sc = scenes.random_block(n_cells=(6, 5, 5), mesh_cells=mesh, seed=seed, vel=2.0, dt=1e-4, stress_scale=2e3,
                                 material=scenes.drucker_prager(psi_deg=5, c=1e3),
                                 bc=scenes.walls(floor=scenes.FREE, sides=scenes.FREE))
        sc["x"] = sc["x"] + np.array([0.0, 0.0, 0.2])
        sc["v"] = sc["v"] + np.asarray(v)
        scs.append(sc)
    ss = [ctx.create_scene(sc, precision=mp.FP64 if prec == "fp64" else mp.FP32) for sc in scs]
    ctx.batch_step(ss, [40, 33])
    for i, (sc, s, k) in enumerate(zip(scs, ss, (40, 33))):
        st = s.stats()
        assert st["error_bits"] == 0 and st["steps_done"] == k and st["n_sorts"] >= 4, (i, st)
        check(f"reorders-large/{mesh}/{prec}/{i}", s.read(), oracle.run(sc, k), sc["x"], BARS[prec])
        s.destroy()


def test_reorders_inside_a_launch_use_the_device(ctx, mp):
    """A small body that reorders every few steps on a mesh of 65536 bricks:
    a step costs about 2.5 times that of the body at rest (reorders by one
    workgroup made it 65 times, separate kernels 2.2 times); 10 leaves room
    for a busy machine."""
    import time
    import torch
    t = []
    for vx in (0.0, 150.0):
        sc = scenes.random_block(n_cells=(8, 8, 8), mesh_cells=(256, 128, 128), seed=7, vel=0.01, dt=1e-4,
                                 gravity=(0.0, 0.0, 0.0), bc=scenes.walls(floor=scenes.FREE, sides=scenes.FREE))
        sc["x"] = sc["x"] + np.array([0.0, 0.0, 0.2])
        sc["v"] = sc["v"] + np.array([vx, 0.3 * vx, 0.2 * vx])
        s = ctx.create_scene(sc, precision=mp.FP32)
        s.step(40)
        best = np.inf
        for _ in range(3):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            s.step(40)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        st = s.stats()
        assert st["error_bits"] == 0 and (st["n_sorts"] > 20) == (vx > 0), st
        t.append(best)
        s.destroy()
    print(f"[reorders-device] per step at rest {t[0] / 40e-6:.1f} us, moving {t[1] / 40e-6:.1f} us", flush=True)
    assert t[1] < 10 * t[0], t


def _spreading(seed=92):
    """10648 particles on 27 bricks that spread over more than 2000."""
    sc = scenes.random_block(n_cells=(11, 11, 11), mesh_cells=(72, 72, 72), seed=seed, vel=0.2, dt=1e-4,
                             gravity=(0.0, 0.0, 0.0), bc=scenes.walls(floor=scenes.FREE, sides=scenes.FREE),
                             material=scenes.elastic(E=1e3), jitter=0.3)
    mid = 36 * sc["mesh"]["h"]
    sc["x"] = sc["x"] - 0.5 * (sc["x"].min(0) + sc["x"].max(0)) + mid
    sc["v"] = sc["v"] + 400.0 * (sc["x"] - mid)
    return sc


def test_a_body_that_has_spread_returns_to_the_separate_kernels(mp):
    """The items that a read reports decide how the next call runs: a body
    that has spread over more than one per compute unit goes back to graphs
    of the separate kernels."""
    sc = _spreading()
    c = mp.Context(0)
    try:
        s = c.create_scene(sc, precision=mp.FP64)
        s.step(100)
        assert c.get_option(mp.OPT_GRAPH_LAUNCHES) == 0
        s.read()
        s.step(17)
        assert c.get_option(mp.OPT_GRAPH_LAUNCHES) == 2
        assert s.stats()["n_items"] > 2000
        check("spread-read", s.read(), oracle.run(sc, 117), sc["x"], BARS["fp64"])
    finally:
        c.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["linear", "gimp", "iso", "slow"])
def test_a_body_that_spreads_within_a_call(ctx, mp, kind, prec):
    """The launch is left within the call, for the wide shape, whose steps
    take more than one launch where the body spreads slowly; scenes that
    spread little or end early go along.  The oracle's location is slow on a
    mesh of this size, so the isoparametric scenes are held against the
    separate kernels (the allocation-free call)."""
    scs = [_spreading(104), scenes.random_block(n_cells=(3, 3, 2), seed=105, vel=0.2, dt=1e-4, gravity=(0.0, 0.0, 0.0),
                                                material=scenes.elastic(E=1e3)),
           scenes.random_block(n_cells=(4, 4, 4), seed=106, vel=0.2, dt=1e-4, gravity=(0.0, 0.0, 0.0),
                               material=scenes.elastic(E=1e3))]
    if kind == "iso":
        scs = [scenes.distort(sc, amp=0.1, seed=107) for sc in scs]
    for sc in scs:
        sc["scheme"]["shape"] = scenes.SHAPE_GIMP if kind == "gimp" else scenes.SHAPE_LINEAR
    k = [110, 90, 110]
    if kind == "slow":
        scs[0]["v"] = 0.5 * scs[0]["v"]
        k = [225, 90, 225]
    ss = [ctx.create_scene(sc, precision=mp.FP64 if prec == "fp64" else mp.FP32) for sc in scs]
    ctx.batch_step(ss, k)
    if kind == "iso":
        other = [ctx.create_scene(sc, precision=mp.FP64) for sc in scs]
        ctx.batch_step_noalloc(other, k)
        refs = [s.read() for s in other]
        for s in other:
            s.destroy()
    else:
        refs = [oracle.run(sc, n) for sc, n in zip(scs, k)]
    for i, (sc, s, ref) in enumerate(zip(scs, ss, refs)):
        st = s.stats()
        assert st["error_bits"] == 0 and st["steps_done"] == k[i], (i, st)
        assert i or st["n_items"] > 2000, st
        check(f"spread-call/{kind}/{prec}/{i}", s.read(), ref, sc["x"], BARS[prec])
        s.destroy()


def test_a_body_that_spreads_costs_little_more_than_in_separate_kernels(mp):
    """100 steps in one call of a body that spreads from 27 to over 2000
    bricks, against the separate kernels: 1.1 times their time (7 times with
    one launch shape and reorders by one workgroup); 3 leaves room for a busy
    machine."""
    import time
    import torch
    sc = _spreading()
    t = []
    for auto in (1, 0):
        c = mp.Context(0)
        c.set_option(mp.OPT_AUTOTUNE, auto)
        best = np.inf
        for _ in range(4):
            s = c.create_scene(sc, precision=mp.FP32)
            s.step(1)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            s.step(100)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
            assert s.stats()["error_bits"] == 0
            s.destroy()
        t.append(best)
        c.close()
    print(f"[spread-time] per step {t[0] * 1e4:.1f} us, separate kernels {t[1] * 1e4:.1f} us", flush=True)
    assert t[0] < 3 * t[1], t


def _iso_body(seed, move):
    """One particle in each cell of a block on a strongly distorted mesh, with
    velocities that move it by up to `move` of a cell per step."""
    h, dt = 0.05, 1e-4
    sc = scenes.random_block(n_cells=(7, 7, 5), mesh_cells=(12, 11, 9), h=h, seed=seed, vel=move * h / dt, dt=dt,
                             material=scenes.elastic(E=1e5), bc=scenes.walls(floor=scenes.FREE, sides=scenes.FREE))
    sc["x"] = sc["x"] + np.array([0.0, 0.0, 2 * h])
    sc.update({k: np.ascontiguousarray(sc[k][seed % 8::8]) for k in ("x", "v", "stress", "vol", "mass")})
    return scenes.distort(sc, amp=0.3, seed=seed + 1)


def _check_nodal_mass(mp, sc, steps):
    """Nodal masses, sums of at most 8 particles' weights here, to 1e-14 of
    the largest: the local coordinates on either side are good to 1.5e-15
    (FP64 rounding), three axes to a weight."""
    c = mp.Context(0)
    try:
        s = c.create_scene(sc, precision=mp.FP64)
        s.step(steps)
        got, ref = s.nodes()["m"], oracle.run(sc, steps)["grid"].m
        err = np.max(np.abs(got - ref)) / np.max(ref)
        print(f"[iso-mass] err {err:.2e}", flush=True)
        assert err <= 1e-14, err
    finally:
        c.close()


@pytest.mark.parametrize("move", [1e-6, 1e-3, 1e-2, 5e-2])
def test_isoparametric_place_of_moved_particles_ends_at_rounding(mp, move):
    """The second step's nodal masses, scattered from the place found for each
    moved particle, whose iteration starts from its old place."""
    for seed in (110, 112, 114):
        _check_nodal_mass(mp, _iso_body(seed, move), 2)


def test_isoparametric_place_on_a_cell_axis_ends_at_rounding(mp):
    """Particles on the axes through their cells' centres, where the first
    guess is exact along the axis but the step matrix is not."""
    for seed in (116, 118, 120):
        sc = _iso_body(seed, 0.0)
        rng = np.random.default_rng(seed)
        mesh, n = sc["mesh"], len(sc["x"])
        X = np.asarray(mesh["node_x"]).reshape(mesh["n"][2] + 1, mesh["n"][1] + 1, mesh["n"][0] + 1, 3)
        r = np.full((n, 3), 0.5)
        r[np.arange(n), rng.integers(0, 3, n)] = rng.uniform(0.03, 0.97, n)
        c = oracle.locate(mesh, sc["x"]).reshape(n, -1)
        if c.shape[1] == 1:
            c = np.stack([c[:, 0] % mesh["n"][0], c[:, 0] // mesh["n"][0] % mesh["n"][1],
                          c[:, 0] // (mesh["n"][0] * mesh["n"][1])], axis=1)
        x = np.zeros((n, 3))
        for q in range(8):
            o = np.array([q & 1, q >> 1 & 1, q >> 2])
            i = c + o
            x += np.prod(np.where(o, r, 1 - r), axis=1)[:, None] * X[i[:, 2], i[:, 1], i[:, 0]]
        sc["x"] = x
        _check_nodal_mass(mp, sc, 1)


@pytest.mark.parametrize("exponent", [-50, -42, 42, 50])
def test_isoparametric_meshes_of_any_unit_of_length(mp, exponent):
    """Cells of 1e-14 to 1e14: the scene scaled by a power of two, whose
    results are those of the original, scaled."""
    sc = _iso_body(122, 0.02)
    L = 2.0 ** exponent
    mesh, mat, sch = dict(sc["mesh"]), dict(sc["material"]), dict(sc["scheme"])
    mesh.update(h=L * mesh["h"], node_x=L * np.asarray(mesh["node_x"]), origin=tuple(L * o for o in mesh["origin"]))
    mat["rho"] = mat["rho"] / L ** 2
    sch["gravity"] = tuple(L * g for g in sch["gravity"])
    big = dict(sc, mesh=mesh, material=mat, scheme=sch, x=L * sc["x"], v=L * sc["v"], vol=L ** 3 * sc["vol"],
               mass=L * sc["mass"])
    ref = oracle.run(sc, 4)
    c = mp.Context(0)
    try:
        s = c.create_scene(big, precision=mp.FP64)
        s.step(4)
        got = s.read()
        check(f"iso-unit/{exponent}", {"x": got["x"] / L, "stress": got["stress"]}, ref, sc["x"], BARS["fp64"])
    finally:
        c.close()


def test_calls_of_few_steps_cost_no_more_than_in_separate_kernels(mp):
    """Calls of three steps of a small linear body, against the separate
    kernels: as much (1.24 times their time in a launch of their own, which
    costs more than two steps save)."""
    import time
    import torch
    sc = scenes.random_block(n_cells=(16, 16, 16), mesh_cells=(36, 36, 36), seed=7, vel=0.01, dt=1e-5,
                             gravity=(0.0, 0.0, 0.0), bc=scenes.walls(floor=scenes.FREE, sides=scenes.FREE))
    c = [mp.Context(0), mp.Context(0)]
    c[1].set_option(mp.OPT_AUTOTUNE, 0)
    ss = [x.create_scene(sc, precision=mp.FP32) for x in c]
    t = [[], []]
    for k in range(300):
        for i in (0, 1):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ss[i].step(3)
            torch.cuda.synchronize()
            t[i].append(time.perf_counter() - t0)
    t = [float(np.median(a)) for a in t]
    print(f"[few-steps] {t[0] * 1e6:.1f} us, separate kernels {t[1] * 1e6:.1f} us", flush=True)
    for x in c:
        x.close()
    assert t[0] < 1.15 * t[1], t


def test_two_contexts_at_once_share_the_device(mp):
    """Two small bodies stepped from two threads at once take no longer than
    with the separate kernels (1.2 times as long where each launch takes every
    compute unit, 0.7 times where it takes what it needs)."""
    import threading
    import time
    sc = scenes.random_block(n_cells=(16, 16, 16), mesh_cells=(36, 36, 36), seed=7, vel=0.01, dt=1e-5,
                             gravity=(0.0, 0.0, 0.0), bc=scenes.walls(floor=scenes.FREE, sides=scenes.FREE))
    t = []
    for auto in (1, 0):
        cs = [mp.Context(0) for _ in range(2)]
        ss = []
        for c in cs:
            c.set_option(mp.OPT_AUTOTUNE, auto)
            ss.append(c.create_scene(sc, precision=mp.FP32))
            ss[-1].step(60)
            ss[-1].read()
        meet = threading.Barrier(3)

        def work(s):
            meet.wait()
            for _ in range(30):
                s.step(100)
                s.read()
            meet.wait()

        th = [threading.Thread(target=work, args=(s,)) for s in ss]
        for x in th:
            x.start()
        meet.wait()
        t0 = time.perf_counter()
        meet.wait()
        t.append(time.perf_counter() - t0)
        for x in th:
            x.join()
        for c in cs:
            c.close()
    print(f"[two-contexts] {t[0] / 30e-6:.0f} us, separate kernels {t[1] / 30e-6:.0f} us", flush=True)
    assert t[0] < 1.1 * t[1], t


def test_reading_one_field_reads_that_field(ctx, mp):
    """A read of the volumes alone of 4.2M particles takes 0.18 times a read
    of everything (0.57 times when every field is loaded)."""
    import time
    import torch
    sc = scenes.random_block(n_cells=(128, 64, 64), mesh_cells=(136, 72, 72), seed=7, vel=0.01, dt=1e-6, jitter=0.1)
    n = len(sc["x"])
    s = ctx.create_scene(sc, precision=mp.FP64)
    s.step(1)
    bufs = {k: torch.empty(v, dtype=torch.int32 if k == "cell" else torch.float64, device="cuda")
            for k, v in dict(x=(n, 3), v=(n, 3), stress=(n, 6), vol=(n,), cell=(n,)).items()}
    t = []
    for fields in (("vol",), tuple(bufs)):
        best = np.inf
        for _ in range(30):
            t0 = time.perf_counter()
            s.read(device_out={k: bufs[k] for k in fields})
            best = min(best, time.perf_counter() - t0)
        t.append(best)
    print(f"[read-one] vol {t[0] * 1e6:.1f} us, everything {t[1] * 1e6:.1f} us", flush=True)
    assert t[0] < 0.38 * t[1], t
    s.destroy()


def test_bodies_that_spread_in_two_contexts_at_once(mp):
    """Two contexts whose launches both outgrow their workgroups and go on in
    the wide shape, each with whatever part of the device the other leaves."""
    import threading
    scs = [_spreading(108), _spreading(109)]
    refs = [oracle.run(sc, 105) for sc in scs]
    out = [None, None]

    def work(i):
        c = mp.Context(0)
        s = c.create_scene(scs[i], precision=mp.FP64)
        for n in (60, 45):
            s.step(n)
        out[i] = (s.read(), s.stats())
        s.destroy()
        c.close()

    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for i in range(2):
        got, st = out[i]
        assert st["error_bits"] == 0 and st["steps_done"] == 105 and st["n_items"] > 1500, st
        check(f"spread-threads/{i}", got, refs[i], scs[i]["x"], BARS["fp64"])
