"""GPU: framed steps of one-field 2D lattices (update, x kernel with the frame,
back into the state) against the FP64 oracle: one line per wave and several,
lines of several waves, grouped and tiled exchange rows, frames that cover a
whole row, single sites and the last one, linear models without products."""

import numpy as np
import pytest

import paper_2405_02410_amd as pss
from oracle import model as om
from oracle.spectral import Lattice as OLattice

pytestmark = pytest.mark.gpu


def _sites(nx, ny):
    row = np.arange(nx) + (ny // 2) * nx          # a whole row
    col = np.arange(ny) * nx + 3                  # a column
    return np.unique(np.concatenate([row, col, [0, nx * ny - 1, 5 * nx + nx - 1]]))


@pytest.mark.parametrize("n,tune", [((16, 16), {}), ((16, 16), {"tc": 1}), ((64, 32), {}), ((32, 512), {}),
                                    ((256, 64), {"px": 8}), ((1024, 16), {}), ((16, 1024), {}), ((4096, 8), {}),
                                    ((8, 4096), {}), ((2048, 16), {})])
def test_fused_frame_steps(n, tune):
    sites = _sites(*n)
    vals = (0.1 * np.cos(np.arange(sites.size))).astype(np.float32)
    lat = pss.Lattice(n, dt=0.01, seed=5)
    lat.tune(**tune)
    f, _ = pss.model_b(lat, D=0.01)
    lat.init_uniform(f, -0.1, 0.1)
    lat.frame(f, sites, vals)
    lat.step(4)
    m = om.model_b(OLattice(*n), 0.01, a=-1.0, b=1.0, k=1.0, D=0.01, seed=5)
    m.init_uniform(0, -0.1, 0.1)
    m.set_frame(0, sites, vals)
    m.step(4)
    got = lat.download(f)
    # 4 steps of four transforms each, ~5e-7 of the framed |phi| <= 0.2 apiece
    assert np.max(np.abs(got - m.real(0).reshape(got.shape))) <= 4e-6


# the step graphs built before any step is taken (prepare) change nothing: the
# first step still forms the products of the uploaded state, on every route of
# a framed step
@pytest.mark.parametrize("n", [(64, 32), (1024, 16), (16, 16, 16), (96, 64), (24, 12, 16), (64,), (60,)])
@pytest.mark.parametrize("fields", [1, 2])
def test_framed_steps_after_prepare(n, fields):
    nx = n[0]
    sites = np.array([i for i in range(int(np.prod(n))) if i % nx < 2])
    rng = np.random.default_rng(3)
    first, second = (rng.uniform(-0.1, 0.1, tuple(reversed(n))).astype(np.float32) for _ in range(2))

    def run(prepare):
        lat = pss.Lattice(n, dt=0.01, seed=5)
        f, _ = pss.model_b(lat, D=0.01)
        if fields == 2:
            g = lat.field("psi")
            lat.term(g, [pss.Mono(-1.0, q2=1)], [(g, 1)], implicit=True)
            lat.term(g, [pss.Mono(-0.3)], [(f, 1), (g, 1)])
            lat.upload(g, second)
        lat.frame(f, sites, np.full(sites.size, 0.2, dtype=np.float32))
        out = []
        for x, k in ((first, 1), (second, 3), (first, 52)):
            lat.upload(f, x)
            if prepare:
                lat.prepare(k)
            lat.step(k)
            out.append(lat.spectrum(f))
        return out

    for a, b in zip(run(True), run(False)):
        assert np.array_equal(a, b)
