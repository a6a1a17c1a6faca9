"""Launches of register tiles: what they read between the calls that move a state."""
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
