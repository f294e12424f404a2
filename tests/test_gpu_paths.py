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
