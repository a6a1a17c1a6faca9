"""Several steps in one launch against the one-step reference kernels, bit for bit.

A call of n steps is dealt to launches of several steps: of tiles held in registers on small grids
(kernel "auto"), else of the fused sweep (which kernel "sweep" asks for).  The state after it, and
the buffer it lies in, are those of n single steps for every n, on grids whose widths and heights
leave partial strips, bands shorter than the rows a fused launch reads beyond them, and halo rows
that wrap around the grid."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1803_00437_amd as F

    F.load_library()
    return F


MRT_SHAPES = [(8, 8), (9, 13), (64, 4), (250, 45), (496, 17), (263, 8), (1021, 70), (37, 300), (240, 130)]


@pytest.mark.parametrize("kernel", ["auto", "sweep"])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("bc", ["periodic", "walls"])
@pytest.mark.parametrize("nx,ny", MRT_SHAPES)
def test_mrt_steps_in_one_launch_equal_reference(F, nx, ny, bc, dtype, kernel):
    if bc == "periodic" and ny < 8:
        pytest.skip("periodic grids have at least eight rows")
    init = W.random_state(nx, ny, seed=nx + ny, amp=0.02)
    kw = dict(scheme="mrt", dtype=dtype, bc=bc, s_xx=1.3, s_e=1.1, s_eps=1.2, s_q=1.4, force=(2e-5, -1e-5))
    ref = F.FdLbm(nx, ny, kernel="reference", **kw)
    got = F.FdLbm(nx, ny, kernel=kernel, **kw)
    ref.set_state(*init)
    got.set_state(*init)
    for n in (3, 1, 2, 4, 5, 8, 14, 37):
        print(f"  mrt {kernel} {nx}x{ny} {bc} {dtype} +{n}", flush=True)
        ref.step(n)
        got.step(n)
        assert got.steps == ref.steps
        assert np.array_equal(got.get_populations(), ref.get_populations())
        # the documented buffer: state_a after an even number of steps since creation
        name = "state_b" if got.steps % 2 else "state_a"
        assert bool((getattr(got.buffers, name) == getattr(ref.buffers, name)).all())
    got.close()
    ref.close()


@pytest.mark.parametrize("dtype,nx,ny", [("f32", 1501, 1600), ("f32", 2600, 905), ("f64", 1203, 1000), ("f64", 998, 1300)])
@pytest.mark.parametrize("bc", ["periodic", "walls"])
def test_mrt_five_steps_in_one_launch_equal_reference(F, nx, ny, dtype, bc):
    """States past the size from which a launch takes five steps."""
    init = W.random_state(nx, ny, seed=nx, amp=0.02)
    kw = dict(scheme="mrt", dtype=dtype, bc=bc, s_xx=1.6, s_e=1.1, quartic=True, force=(1e-5, 2e-5))
    ref = F.FdLbm(nx, ny, kernel="reference", **kw)
    got = F.FdLbm(nx, ny, **kw)
    assert got.state_bytes >= 80 << 20
    ref.set_state(*init)
    got.set_state(*init)
    for n in (5, 11, 7):
        print(f"  mrt fused {nx}x{ny} {bc} {dtype} +{n}", flush=True)
        ref.step(n)
        got.step(n)
        name = "state_b" if got.steps % 2 else "state_a"
        assert bool((getattr(got.buffers, name) == getattr(ref.buffers, name)).all())
    got.close()
    ref.close()


FD_SHAPES = [(8, 8), (9, 13), (64, 12), (250, 45), (240, 17), (263, 9), (502, 16), (1021, 70), (37, 300), (480, 130)]
FD_KINDS = [("fd", 3, "periodic", 0.5), ("fd", 3, "walls", 0.5), ("fd", 3, "walls", 0.8), ("fd", 5, "periodic", 0.5), ("lwacm", 3, "periodic", 0.5)]


@pytest.mark.parametrize("kernel", ["auto", "sweep"])
@pytest.mark.parametrize("dtype", ["f32", "f64", "f16", "f16sr"])
@pytest.mark.parametrize("scheme,stencil,bc,xi", FD_KINDS)
@pytest.mark.parametrize("forced", [False, True])
@pytest.mark.parametrize("nx,ny", FD_SHAPES)
def test_fd_steps_in_one_launch_equal_reference(F, nx, ny, scheme, stencil, bc, xi, dtype, forced, kernel):
    if forced and scheme == "lwacm":
        pytest.skip("the LW-ACM step has no body force")
    init = W.random_state(nx, ny, seed=nx + ny, amp=0.02)
    kw = dict(scheme=scheme, dtype=dtype, bc=bc, s_xx=1.3, s_e=1.1)
    if scheme == "fd":
        kw.update(stencil=stencil, wall_xi=xi, force=(2e-5, -1e-5) if forced else (0.0, 0.0))
    ref = F.FdLbm(nx, ny, kernel="reference", **kw)
    got = F.FdLbm(nx, ny, kernel=kernel, **kw)
    ref.set_state(*init)
    got.set_state(*init)
    for n in (3, 1, 2, 4, 8, 21):
        print(f"  {scheme}{stencil} {kernel} {nx}x{ny} {bc} xi {xi} {dtype} +{n}", flush=True)
        ref.step(n)
        got.step(n)
        name = "state_b" if got.steps % 2 else "state_a"
        assert got.steps == ref.steps
        assert bool((getattr(got.buffers, name) == getattr(ref.buffers, name)).all())
    got.close()
    ref.close()


DISKS = [(72, 72, (35.5, 35.5, 29.9)), (50, 41, (24.3, 19.8, 11.7)), (300, 200, (149.5, 99.5, 80.0))]


@pytest.mark.parametrize("dtype", ["f32", "f64", "f16", "f16sr"])
@pytest.mark.parametrize("scheme,stencil,force", [("fd", 3, 0.0), ("fd", 5, 0.0), ("fd", 3, 2e-5), ("lwacm", 3, 0.0)])
@pytest.mark.parametrize("nx,ny,disk", DISKS)
def test_disk_fill_and_step_in_one_launch_equal_reference(F, nx, ny, disk, scheme, stencil, force, dtype):
    init = W.random_state(nx, ny, seed=nx, amp=2e-3)
    kw = dict(scheme=scheme, dtype=dtype, bc="disk", disk=disk, s_xx=1.3, s_e=1.1)
    if scheme == "fd":
        kw.update(stencil=stencil, force=(force, -force))
    ref = F.FdLbm(nx, ny, kernel="reference", **kw)
    got = F.FdLbm(nx, ny, **kw)
    for start in (0, 7):  # a state set again finds the rest nodes of the last run
        ref.set_state(*init)
        got.set_state(*init)
        for n in (1, 2, 5):
            print(f"  disk {scheme}{stencil} {nx}x{ny} {dtype} from {start} +{n}", flush=True)
            ref.step(n)
            got.step(n)
            assert all(np.array_equal(a, b) for a, b in zip(got.get_state(), ref.get_state()))
    got.close()
    ref.close()


@pytest.mark.parametrize("dtype", ["f32", "f64", "f16"])
def test_batch_steps_in_one_launch_equal_reference(F, dtype):
    """Widths around the strips of two and three steps (116, 120 and 52, 56 columns), odd and even."""
    sizes = [(8, 8), (9, 30), (52, 9), (57, 120), (115, 11), (116, 64), (121, 45), (123, 123), (124, 17), (129, 8),
             (236, 33), (239, 70), (241, 240), (512, 100)]
    specs = [(nx, ny, 1.2 + 0.01 * i, 1.1) for i, (nx, ny) in enumerate(sizes)]
    batch = F.FdLbmBatch(specs, dtype=dtype, max_samples=4)
    refs = []
    for i, (nx, ny, s_xx, s_e) in enumerate(specs):
        init = W.random_state(nx, ny, seed=i, amp=0.02)
        batch.set_state(i, *init)
        refs.append(F.FdLbm(nx, ny, dtype=dtype, s_xx=s_xx, s_e=s_e, kernel="reference"))
        refs[-1].set_state(*init)
    for n, every in ((1, 0), (2, 0), (5, 0), (10, 5), (7, 7), (13, 0)):
        print(f"  batch {dtype} +{n} every {every}", flush=True)
        batch.step(n, sample_every=every)
        batch.stream.synchronize()
        for i, ref in enumerate(refs):
            ref.step(n)
            assert all(np.array_equal(a, b) for a, b in zip(batch.get_state(i), ref.get_state())), sizes[i]
    batch.close()
    for ref in refs:
        ref.close()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nx,ny,nz", [(3, 3, 3), (61, 11, 5), (64, 10, 2 * 37 + 1), (120, 21, 130), (256, 130, 9)])
def test_d3_planes_chosen_from_the_grid_equal_reference(F, nx, ny, nz, dtype):
    """The default planes per block: one block of planes, uneven ones, and the smallest grid."""
    init = W.random_state3(nx, ny, nz, seed=nx + nz, amp=0.02)
    kw = dict(dtype=dtype, s_nu=1.4, s_e=1.2)
    ref = F.FdLbm3D(nx, ny, nz, kernel="reference", **kw)
    got = F.FdLbm3D(nx, ny, nz, **kw)
    ref.set_state(*init)
    got.set_state(*init)
    print(f"  d3 {nx}x{ny}x{nz} {dtype}", flush=True)
    ref.step(5)
    got.step(5)
    size = 4 * nx * ny * nz * (8 if dtype == "f64" else 4)  # the buffers are padded to 256 bytes
    assert bool((got.buffers.state_b[:size] == ref.buffers.state_b[:size]).all())
    got.close()
    ref.close()


def test_diagnostics_of_many_contexts(F):
    """More contexts than there are pinned result slots: every one reads its own numbers."""
    sims = []
    for i in range(70):
        sim = F.FdLbm(16, 8, dtype="f64", s_xx=1.2)
        sim.set_state(np.full((8, 16), 1e-3 * i), np.zeros((8, 16)), np.zeros((8, 16)))
        sims.append(sim)
    for _ in range(5):  # copied at first, then written to a slot
        for i, sim in enumerate(sims):
            assert sim.diagnostics()["mass"] == pytest.approx(128 * 1e-3 * i, abs=1e-12)
    for sim in sims[::2]:
        sim.close()
    again = F.FdLbm(16, 8, dtype="f64", s_xx=1.2)
    again.set_state(np.full((8, 16), 0.5), np.zeros((8, 16)), np.zeros((8, 16)))
    for _ in range(5):
        assert again.diagnostics()["mass"] == pytest.approx(64.0)
    assert sims[1].diagnostics()["mass"] == pytest.approx(0.128)
    for sim in sims[1::2] + [again]:
        sim.close()


@pytest.mark.parametrize("nx,ny,n,kw", [
    (72, 72, 10, dict(dtype="f64", bc="disk", disk=(35.5, 35.5, 29.9))),
    (64, 64, 10, dict(dtype="f64")),
    (1030, 520, 8, dict(dtype="f32", kernel="sweep")),
    (191, 100, 12, dict(dtype="f64", scheme="lwacm")),
    (333, 200, 10, dict(dtype="f32", scheme="mrt")),
])
def test_recorded_steps_replay(F, nx, ny, n, kw):
    """Steps recorded into a graph, which then runs on another stream, with the state read (through
    the staging area) between its replays: the bits of the same steps issued one call at a time."""
    import torch

    init = W.random_state(nx, ny, seed=3, amp=2e-3)
    eager = F.FdLbm(nx, ny, s_xx=1.3, s_e=1.1, **kw)
    sim = F.FdLbm(nx, ny, s_xx=1.3, s_e=1.1, stream=torch.cuda.Stream(), **kw)
    for s in (eager, sim):
        s.set_state(*init)
        s.step(n)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=sim.stream):
        sim.step(n)
    for r in range(3):
        print(f"  replay {r} of {nx}x{ny} {kw}", flush=True)
        graph.replay()
        torch.cuda.synchronize()
        eager.step(n)
        assert all(np.array_equal(a, b) for a, b in zip(sim.get_state(), eager.get_state()))
    eager.close()
    sim.close()
