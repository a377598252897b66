"""Host check of a model's stability (no GPU): what pss_validate accepts and
refuses equals an evaluation at every mode, on both sides of the limit, for
operators that its bounds decide and for those that it has to evaluate."""

import numpy as np
import pytest

import paper_2405_02410_amd as pss
from paper_2405_02410_amd import Mono, PssError


def _q2(n, dx):
    q2 = np.zeros((1,) * len(n))
    for i, (m, d) in enumerate(zip(n, dx)):
        k = np.fft.fftfreq(m, d) * 2 * np.pi
        q2 = q2 + (k ** 2).reshape([-1 if j == i else 1 for j in range(len(n))])
    return q2


@pytest.mark.parametrize("n,dx", [((64,), (0.7,)), ((16, 32), (1.0, 0.5)), ((12, 10), (1.0, 2.0)), ((8, 16, 8), (1.0, 1.5, 0.8))])
@pytest.mark.parametrize("op", [[(1.0, 1)], [(1.0, 1), (-1.0, 2)], [(1.0, 0), (2.0, 1), (-0.5, 2), (0.01, 3)], [(-1.0, 1)],
                                [(0.3, 0)], [(-4.0, 0), (4.0, 1), (-1.0, 2)]])
def test_validate_decides_as_every_mode_does(n, dx, op):
    q2 = _q2(n, dx)
    top = max(np.max(sum(c * q2 ** p for c, p in op)), 0.0)
    limit = 1.0 / top if top > 0 else None  # refused from this dt on
    dts = [1e-3, 10.0] if limit is None else [limit * f for f in (1e-3, 0.5, 0.99, 0.9999, 1 - 1e-9, 1 + 1e-9, 1.01, 10.0)]
    for dt in dts:
        lat = pss.Lattice(n, dx=dx, dt=dt)
        f = lat.field("phi")
        lat.term(f, [Mono(c, q2=p) for c, p in op], [(f, 1)], implicit=True)
        lat.noise(f, [Mono(0.1, q2=1), Mono(0.0)])
        if limit is not None and dt >= limit:
            with pytest.raises(PssError) as e:
                lat.validate()
            assert e.value.name == "PSS_E_UNSTABLE"
        else:
            lat.validate()


def test_noise_that_is_negative_somewhere_only():
    for coef, ok in ((0.01, True), (-0.01, False)):
        lat = pss.Lattice((16, 16), dt=0.01)
        f, _ = pss.model_b(lat, D=0.0)
        lat.noise(f, [Mono(0.05, q2=1), Mono(coef, q2=2)])
        if ok:
            lat.validate()
        else:
            with pytest.raises(PssError) as e:
                lat.validate()
            assert e.value.name == "PSS_E_INVAL"
