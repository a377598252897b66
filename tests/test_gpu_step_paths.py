"""GPU: the forms that a step's launches take by size (exchange arrays in
groups of four rows or in column tiles, the self-conjugate modes of a packed
line in four lanes or in one thread, 3D points per thread), each against the
FP64 oracle, and regroupings of the same arithmetic against each other."""

import numpy as np
import pytest

import paper_2405_02410_amd as pss
from oracle import model as om
from oracle.spectral import Lattice as OLattice

pytestmark = pytest.mark.gpu


def _run(n, steps, **tune):
    lat = pss.Lattice(n, dt=0.01, seed=11)
    lat.tune(**tune)
    f, _ = pss.model_b(lat, a=-1.0, b=1.0, k=1.0, D=0.01)
    lat.init_uniform(f, -0.1, 0.1)
    lat.step(steps)
    return lat.spectrum(f), lat.download(f)


def _oracle(n, steps):
    m = om.model_b(OLattice(*n), 0.01, a=-1.0, b=1.0, k=1.0, D=0.01, seed=11)
    m.init_uniform(0, -0.1, 0.1)
    m.step(steps)
    return m.real(0).reshape(tuple(reversed(n)))


# lines of 8 (two threads: no groups, the self-conjugate modes in one thread),
# 16 (four threads: the smallest line in groups), one wave and several
@pytest.mark.parametrize("n", [(8, 8), (16, 8), (8, 16), (16, 16), (64, 16), (16, 64), (64, 256), (32, 1024)])
def test_one_column_tiles_equal_wider_tiles_and_the_oracle(n):
    pu = {"pu": 8} if n[1] == 1024 else {}  # two lines of 1024 in a block take 8 points per thread
    tall, real = _run(n, 5, tc=1, **pu)
    wide, _ = _run(n, 5, tc=2, **pu)
    assert np.array_equal(tall, wide)
    # 5 steps at ~2e-6 of |phi| <= 0.1 each
    assert np.max(np.abs(real - _oracle(n, 5))) <= 2e-6


# points per thread change the radix and so the rounding: 1e-5 of |phi| <= 0.1
@pytest.mark.parametrize("n", [(16, 16, 16), (16, 32, 64), (32, 256, 16)])
def test_3d_points_per_thread(n):
    want = _oracle(n, 3)
    for tune in ({}, {"pu": 8, "px": 8, "py": 8}, {"pu": 8, "py": 16, "tz": 1}):
        _, real = _run(n, 3, **tune)
        assert np.max(np.abs(real - want)) <= 2e-6, tune


# lines of 2048 and 4096: one guarded block buffer, split twiddles, blocks of
# 512 threads, in either direction, and the forms that 16 points a thread keep
@pytest.mark.parametrize("n", [(2048, 16), (16, 2048), (4096, 8), (8, 4096)])
def test_long_lines(n):
    want = _oracle(n, 5)
    for tune in ({}, {"pu" if n[1] > n[0] else "px": 16}):
        _, real = _run(n, 5, **tune)
        assert np.max(np.abs(real - want)) <= 2e-6, tune


# mixed-radix steps on half spectra: odd line pairs, every radix of the passes
# (2 3 4 5 6 8 9 10 12 15 16 among these sizes), blocks of one and two lines
# with a ragged last block, and no de-aliasing (column Nx/2 is kept)
@pytest.mark.parametrize("n", [(12, 10), (18, 50), (162, 20), (90, 96), (240, 30), (10, 2048), (1500, 12), (24, 10, 18),
                               (16, 30, 12), (800, 12, 8)])
@pytest.mark.parametrize("dealias", [pss.DEALIAS_TWO_THIRDS, pss.DEALIAS_NONE])
def test_mixed_radix_steps(n, dealias):
    lat = pss.Lattice(n, dt=0.01, seed=11, dealias=dealias)
    f, _ = pss.model_b(lat, a=-1.0, b=1.0, k=1.0, D=0.01)
    lat.init_uniform(f, -0.1, 0.1)
    lat.step(5)
    rule = {pss.DEALIAS_TWO_THIRDS: om.DEALIAS_TWO_THIRDS, pss.DEALIAS_NONE: om.DEALIAS_NONE}[dealias]
    m = om.model_b(OLattice(*n), 0.01, a=-1.0, b=1.0, k=1.0, D=0.01, seed=11, dealias=rule)
    m.init_uniform(0, -0.1, 0.1)
    m.step(5)
    got = lat.download(f)
    assert np.max(np.abs(got - m.real(0).reshape(got.shape))) <= 2e-6


# the adjoint's column launches: lines of two and four threads, one wave and
# several, tiles of one and more columns, segments of one step, of several and
# a shorter last one; the bar is that of the adjoint's own tests (1e-3)
@pytest.mark.parametrize("n,ckpt", [((16, 8), 1), ((8, 16), 4), ((16, 256), 5), ((16, 1024), 11), ((256, 32), 20)])
def test_adjoint_line_forms(n, ckpt):
    from tests.test_gpu_adjoint import _check, _gpu, _oracle as adjoint_oracle

    S_star, Lo, go, gphio = adjoint_oracle(n, 11, seed=5)
    lat = _gpu(n, seed=5)
    L, g, gphi = lat.adjoint_model_b(11, S_star, ckpt_every=ckpt)
    _check(L, g, gphi, Lo, go, gphio)
    twin = _gpu(n, seed=5)
    twin.step(11)
    assert lat.step_index == 11 and np.array_equal(lat.spectrum(0), twin.spectrum(0))


# lines stepped on half spectra: every length's threads and waves, both ends of
# the spectrum kept (no de-aliasing), two products in one channel, more steps
# than the mode N/2 draws at once (64), and the same in two chunks
@pytest.mark.parametrize("n", [8, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("dealias", [pss.DEALIAS_TWO_THIRDS, pss.DEALIAS_NONE])
def test_half_spectrum_lines(n, dealias):
    def make(chunks):
        lat = pss.Lattice((n,), dt=0.01, seed=11, dealias=dealias)
        f = lat.field("phi")
        lat.term(f, [pss.Mono(1.0, q2=1), pss.Mono(-1.0, q2=2)], [(f, 1)], implicit=True)
        lat.term(f, [pss.Mono(-1.0, q2=1)], [(f, 3)])
        lat.term(f, [pss.Mono(-1.0, q2=1)], [(f, 2)])
        lat.noise(f, [pss.Mono(0.01, q2=1), pss.Mono(0.01)])
        lat.init_uniform(f, -0.1, 0.1)
        for k in chunks:
            lat.step(k)
        return lat.spectrum(f), lat.download(f)

    rule = {pss.DEALIAS_TWO_THIRDS: om.DEALIAS_TWO_THIRDS, pss.DEALIAS_NONE: om.DEALIAS_NONE}[dealias]
    m = om.Model(OLattice(n), 0.01, seed=11, dealias=rule)
    f = m.add_field("phi")
    m.add_term(f, [om.Mono(1.0, q2=1), om.Mono(-1.0, q2=2)], [(f, 1)], implicit=True)
    m.add_term(f, [om.Mono(-1.0, q2=1)], [(f, 3)])
    m.add_term(f, [om.Mono(-1.0, q2=1)], [(f, 2)])
    m.set_noise(f, [om.Mono(0.01, q2=1), om.Mono(0.01)])
    m.init_uniform(f, -0.1, 0.1)
    m.step(70)
    sp, real = make([70])
    # as the other 1D parity runs: 1e-4 of max(1, |phi|) after some 100 steps
    want = m.real(f)[0, 0]
    assert np.max(np.abs(real - want)) <= 1e-4 * max(1.0, np.max(np.abs(want)))
    ws = m.state[f][0, 0, : n // 2 + 1]
    assert np.max(np.abs(sp - ws)) <= 1e-4 * np.max(np.abs(ws))
    sp2, _ = make([33, 37])
    assert np.array_equal(sp, sp2)


# a batch after its members' own work: downloaded (nothing left on the member's
# stream) and stepped alone (work left on it), one on a caller's stream
def test_batch_orders_itself_after_downloads_and_steps():
    import torch

    def members():
        lats = []
        for i, n in enumerate([64, 64, 128, 256]):
            lat = pss.Lattice((n, n), dt=0.01, seed=20 + i)
            f, _ = pss.model_b(lat, D=0.01)
            lat.init_uniform(f, -0.1, 0.1)
            lats.append((lat, f))
        return lats

    lats, alone = members(), members()
    stream = torch.cuda.Stream()
    lats[1][0].stream(stream.cuda_stream)
    batch = pss.Batch([lat for lat, _ in lats])
    outs = [torch.empty(lat.shape, device="cuda") for lat, _ in lats]
    for k in range(3):
        batch.step(7)
        for (lat, f), out in zip(lats, outs):
            lat.download(f, out)
        for (lat, _), out in zip(lats[::2], outs):
            lat.step(120)
        batch.step(5)
        lats[1][0].download(lats[1][1], outs[1])
    for i, (lat, f) in enumerate(alone):
        for k in range(3):
            lat.step(7)
            if i % 2 == 0:
                lat.step(120)
            lat.step(5)
    for (lat, f), (one, g) in zip(lats, alone):
        assert np.array_equal(lat.spectrum(f), one.spectrum(g))


# downloads into device memory written in place of a copy: a whole tensor, a
# part of one at any offset, and host tensors, which are copied to
@pytest.mark.parametrize("n", [(16,), (60,), (32, 16), (24, 20), (16, 8, 8)])
def test_downloads_into_tensors(n):
    import torch

    lat = pss.Lattice(n, dt=0.01, seed=3)
    f, _ = pss.model_b(lat, D=0.01)
    lat.init_uniform(f, -0.1, 0.1)
    lat.step(3)
    want = lat.download(f)
    for dev in ("cuda", "cpu"):
        for off in (0, 1, 3, 64):
            big = torch.full((want.size + 100,), 7.0, device=dev)
            torch.cuda.synchronize()
            lat.download(f, big[off:off + want.size])
            got = big.cpu().numpy()
            assert np.array_equal(got[off:off + want.size].reshape(want.shape), want)
            assert np.all(got[:off] == 7.0) and np.all(got[off + want.size:] == 7.0)


# the adjoint with every state kept and with checkpoints: the same bits, the
# same lattice afterwards (segments of one step, several, a shorter last one)
@pytest.mark.parametrize("n,steps,ckpt", [((16, 8), 1, 1), ((64, 32), 23, 5), ((32, 1024), 9, 9), ((64, 64), 70, 1)])
def test_adjoint_with_and_without_recomputation(monkeypatch, n, steps, ckpt):
    from tests.test_gpu_adjoint import _gpu

    S = np.full(min(n) // 2 - 1, 0.01)
    got = []
    for whole in ("0", "1"):
        monkeypatch.setenv("PSS_TAPE_WHOLE", whole)
        lat = _gpu(n, seed=5)
        lat.step(2)
        L, g, gphi = lat.adjoint_model_b(steps, S, ckpt_every=ckpt)
        at = lat.step_index, lat.spectrum(0)
        lat.step(3)
        got.append((L, g, gphi, *at, lat.spectrum(0)))
    for x, y in zip(*got):
        assert np.array_equal(x, y)
    twin = _gpu(n, seed=5)
    twin.step(steps + 2)
    assert np.array_equal(twin.spectrum(0), got[0][4])
    twin.step(3)
    assert np.array_equal(twin.spectrum(0), got[0][5])


# lattices that differ in their de-aliasing alone share a class and its
# launches, each with its own kept columns: in LDS, fused, and launched by class
@pytest.mark.parametrize("n,model,launches", [((64, 64), "b", (0, 0, 1)), ((256, 128), "b", (2, 1, 0)),
                                              ((32, 16), "b", (2, 0, 0)), ((128, 64), "kpz", (2, 0, 0))])
def test_batch_of_lattices_that_differ_in_their_dealiasing(n, model, launches):
    def make():
        out = []
        for i, (rule, shape) in enumerate([(pss.DEALIAS_TWO_THIRDS, pss.SHAPE_RADIAL), (pss.DEALIAS_NONE, pss.SHAPE_RADIAL),
                                           (pss.DEALIAS_PAPER_ORDER, pss.SHAPE_PER_AXIS), (pss.DEALIAS_NONE, pss.SHAPE_RADIAL)]):
            lat = pss.Lattice(n, dt=0.01, seed=30 + i, dealias=rule, shape=shape)
            f = pss.model_b(lat, D=0.01)[0] if model == "b" else pss.kpz(lat, D=0.01)[0]
            lat.init_uniform(f, -0.5, 0.5)
            out.append((lat, f))
        return out

    mem, alone = make(), make()
    batch = pss.Batch([lat for lat, _ in mem])
    assert batch.classes() == (1, [0, 0, 0, 0])
    assert batch.launches() == launches
    batch.step(40)
    mem[1][0].step(3)
    batch.step(7)
    for i, ((lat, f), (one, g)) in enumerate(zip(mem, alone)):
        one.step(50 if i == 1 else 47)
        assert np.array_equal(lat.spectrum(f), one.spectrum(g)), i
    batch.close()


# the adjoint over lines of 4096 (blocks of 512 threads in its two launches)
@pytest.mark.parametrize("n", [(4096, 8), (8, 4096)])
def test_adjoint_of_the_longest_lines(n):
    from tests.test_gpu_adjoint import _check, _gpu, _oracle as adjoint_oracle

    S_star, Lo, go, gphio = adjoint_oracle(n, 6, seed=5)
    for ckpt in (0, 1):
        lat = _gpu(n, seed=5)
        lat.tune(ckpt=ckpt)
        L, g, gphi = lat.adjoint_model_b(6, S_star, ckpt_every=4)
        _check(L, g, gphi, Lo, go, gphio)
