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
