"""Launches of register tiles: every compiled shape against the one-step reference kernels, bit for bit,
and what they read between the calls that move a state."""
import functools

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


@pytest.mark.parametrize("scheme,dtype", [("fd", "f64"), ("fd", "f32"), ("lwacm", "f16")])
def test_disk_steps_read_nothing_that_a_state_transfer_writes(F, scheme, dtype):
    """A transfer writes its FP64 planes into the scratch buffer and nothing else there, so steps
    recorded into a graph may run while a state is read: the planes are found whole after
    get_state, and steps after they are overwritten keep the reference's bits."""
    nx, ny = 72, 61
    init = W.random_state(nx, ny, seed=3, amp=2e-3)
    kw = dict(scheme=scheme, dtype=dtype, bc="disk", disk=(35.5, 30.2, 26.3), s_xx=1.3, s_e=1.1)
    ref = F.FdLbm(nx, ny, kernel="reference", **kw)
    got = F.FdLbm(nx, ny, **kw)
    for s in (ref, got):
        s.set_state(*init)
        s.step(3)
    planes = np.concatenate([a.ravel() for a in got.get_state()]).tobytes()
    start = got.buffers.scratch.cpu().numpy().tobytes().find(planes)
    assert start >= 0
    got.buffers.scratch[start:start + len(planes)] = 0x7F
    print(f"  disk {scheme} {nx}x{ny} {dtype}: planes at {start}", flush=True)
    ref.step(5)
    got.step(5)
    assert all(np.array_equal(a, b) for a, b in zip(got.get_state(), ref.get_state()))
    got.close()
    ref.close()


# (kind, dtype, boundary, body force); tests/test_launch_plan.py holds the grids to every shape that a
# plan can give any of them
TILE_KINDS = [(k, d, bc, force) for k, dtypes in (("fd3", ("f64", "f32", "f16", "f16sr")),
                                                  ("fd5", ("f64", "f32", "f16", "f16sr")),
                                                  ("lwacm", ("f64", "f32", "f16", "f16sr")), ("mrt", ("f64", "f32")))
              for d in dtypes for bc, force in (("periodic", 0), ("periodic", 1), ("walls", 1), ("disk", 0))
              if not (k == "lwacm" and (force or bc == "walls")) and not (k == "fd5" and bc == "walls")
              and not (k == "mrt" and bc == "disk")]
TILE_GRIDS = [(17, 20), (373, 376), (615, 618), (681, 684), (879, 882), (945, 948), (967, 970)]
TILE_STEPS = 50


@functools.lru_cache(maxsize=None)
def random_state(nx, ny):
    return W.random_state(nx, ny, seed=nx, amp=2e-3)


@pytest.mark.parametrize("kind,dtype,bc,force", TILE_KINDS)
def test_every_tile_shape_equals_reference(F, kind, dtype, bc, force):
    """Calls of TILE_STEPS steps and of a few, on grids whose last tiles are partly filled."""
    for nx, ny in TILE_GRIDS:
        kw = dict(scheme=kind if kind in ("lwacm", "mrt") else "fd", dtype=dtype, bc=bc, s_xx=1.3, s_e=1.1)
        if kind.startswith("fd"):
            kw["stencil"] = int(kind[2])
        if kind == "mrt":
            kw.update(s_eps=1.2, s_q=1.4)
        if force:
            kw["force"] = (2e-5, -1e-5)
        if bc == "disk":
            kw["disk"] = ((nx - 1) / 2 - 0.2, (ny - 1) / 2 + 0.1, min(nx, ny) / 2 - 3.5)
        ref = F.FdLbm(nx, ny, kernel="reference", **kw)
        got = F.FdLbm(nx, ny, **kw)
        ref.set_state(*random_state(nx, ny))
        got.set_state(*random_state(nx, ny))
        for n in (TILE_STEPS, 9):
            print(f"  {kind} {dtype} {bc} force {force} {nx}x{ny} +{n}", flush=True)
            ref.step(n)
            got.step(n)
            assert all(np.array_equal(a, b) for a, b in zip(got.get_state(), ref.get_state())), (nx, ny, n)
            if kind == "mrt":
                assert np.array_equal(got.get_populations(), ref.get_populations()), (nx, ny, n)
        got.close()
        ref.close()


@pytest.mark.parametrize("bc", ["periodic", "walls"])
@pytest.mark.parametrize("dtype,nx,ny", [("f32", 63, 40), ("f32", 190, 33), ("f32", 191, 20), ("f32", 254, 30),
                                         ("f32", 1022, 9), ("f32", 3003, 2501), ("f64", 191, 20), ("f64", 254, 30),
                                         ("f64", 2001, 1901)])
def test_mrt_single_steps_equal_reference(F, dtype, nx, ny, bc):
    """Widths of one, two and four columns per lane, and states past the last-level cache, whose odd widths
    are read at element-aligned offsets."""
    kw = dict(scheme="mrt", dtype=dtype, bc=bc, s_xx=1.3, s_e=1.1, s_eps=1.2, s_q=1.4, force=(2e-5, -1e-5))
    ref = F.FdLbm(nx, ny, kernel="reference", **kw)
    got = F.FdLbm(nx, ny, kernel="sweep", **kw)
    for s in (ref, got):
        s.set_state(*random_state(nx, ny))
    for n in (1, 2):
        print(f"  mrt {dtype} {bc} {nx}x{ny} +{n}", flush=True)
        for _ in range(n):
            ref.step(1)
            got.step(1)
        name = "state_b" if got.steps % 2 else "state_a"
        assert bool((getattr(got.buffers, name) == getattr(ref.buffers, name)).all())
    got.close()
    ref.close()


def test_d3_autotune_leaves_no_slower_steps(F):
    """A thin grid runs in many blocks of a few planes (8.4 us per step at 8 x 8 x 64), which none of the
    tuner's shapes has (16 planes and more: 25 us and more)."""
    import torch

    sim = F.FdLbm3D(8, 8, 64, dtype="f32", s_nu=1.4, s_e=1.2)
    sim.set_state(*W.random_state3(8, 8, 64, seed=1, amp=0.02))

    def step_us():
        best = 1e9
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            sim.step(50)
            e1.record()
            e1.synchronize()
            best = min(best, 1e3 * e0.elapsed_time(e1) / 50)
        return best

    step_us()
    before = step_us()
    rows, planes, ms = sim.autotune(reps=5)
    after = step_us()
    print(f"  d3 8x8x64: {before:.1f} us, autotune {rows} rows {planes} planes {1e3 * ms:.1f} us, then {after:.1f} us", flush=True)
    assert rows in (8, 12, 16) and planes in (16, 32, 64, 128)
    assert after < 1.7 * before
    sim.close()


def launches(F, n, nx, ny, **kw):
    """Kernel launches that a call of n steps records."""
    import ctypes

    import torch

    sim = F.FdLbm(nx, ny, s_xx=1.3, s_e=1.1, stream=torch.cuda.Stream(), **kw)
    sim.set_state(*random_state(nx, ny))
    sim.step(n)
    torch.cuda.synchronize()
    hip = ctypes.CDLL("libamdhip64.so")
    stream, graph, count = ctypes.c_void_p(sim.stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipStreamBeginCapture(stream, 1) == 0  # thread-local
    sim.step(n)
    assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    hip.hipGraphDestroy(graph)
    sim.close()
    return count.value


@pytest.mark.parametrize("kw", [dict(dtype="f64"), dict(dtype="f32", scheme="mrt"), dict(dtype="f32", scheme="lwacm"),
                                dict(dtype="f32", kernel="sweep")])
def test_one_row_per_tile_is_no_choice(F, kw):
    """tile_rows = 1 leaves the choice to the library, as 0 does; other rows are those of one-step launches."""
    n = [launches(F, 12, 200, 150, tile_rows=rows, **kw) for rows in (0, 1, 4)]
    print(f"  {kw}: launches of 12 steps {n}", flush=True)
    assert n[0] == n[1] < n[2] == 12
