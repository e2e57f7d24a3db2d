"""Where hair_set_cluster_params takes its arrays from: allocations of exactly the array's size and
places inside larger ones are copied, host memory as well, and an array that would run past the end
of its allocation is refused with an error instead of being read."""
import ctypes as C

import numpy as np
import pytest
import torch

import hairsynth as hs

pytestmark = pytest.mark.gpu

K, S = 7, 5          # axes 280 bytes, r 28, sigma_a 84


class _Raw:
    """Device memory of an exact size (torch's own allocations are parts of larger ones).  Every
    case stays below 4 KiB, so all bytes that a copy could touch lie in the allocation's page."""

    def __init__(self):
        torch.zeros(1, device="cuda:0")
        path = {line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line}
        self.hip = C.CDLL(sorted(path)[0])
        self.held = []

    def take(self, nbytes):
        p = C.c_void_p()
        assert self.hip.hipMalloc(C.byref(p), C.c_size_t(nbytes)) == 0
        self.held.append(p)
        return p.value

    def fill(self, ptr, values):
        v = np.ascontiguousarray(values, dtype=np.float32)
        assert self.hip.hipMemcpy(C.c_void_p(ptr), C.c_void_p(v.ctypes.data), C.c_size_t(v.nbytes), 1) == 0

    def close(self):
        self.hip.hipGetLastError()      # (a refused copy's error is the thread's last one)
        for p in self.held:
            self.hip.hipFree(p)


class _At:
    def __init__(self, ptr):
        self.ptr = ptr

    def data_ptr(self):
        return self.ptr


@pytest.fixture()
def level(hip):
    ctx = hip.Context(0)
    asset = hs.make_asset(40, S, 60.0, seed=3)
    aid = ctx.upload_asset(asset)
    ctx.build_lod(aid, [(np.arange(40) % K).astype(np.int32)])
    lod = ctx.get_lod(aid, 1)
    new = [(1.5 * np.array(a) + 1e-4).astype(np.float32) for a in (lod.axes, lod.r, lod.sigma_a)]
    raw = _Raw()
    yield ctx, aid, new, raw
    raw.close()
    ctx.close()


def _stored(ctx, aid):
    lod = ctx.get_lod(aid, 1)
    return [np.array(a) for a in (lod.axes, lod.r, lod.sigma_a)]


@pytest.mark.parametrize("shift", [0, 4, 64])
def test_exact_and_inner_arrays_are_copied(level, shift):
    ctx, aid, new, raw = level
    print(f"case: arrays {shift} bytes into allocations that end with them", flush=True)
    at = []
    for a in new:
        p = raw.take(a.nbytes + shift) + shift
        raw.fill(p, a)
        at.append(_At(p))
    ctx.set_cluster_params(aid, 1, *at)
    torch.cuda.synchronize()
    for got, want in zip(_stored(ctx, aid), new):
        assert np.array_equal(got, want)


def test_host_arrays_are_copied(level):
    ctx, aid, new, _ = level
    print("case: arrays in pinned host memory", flush=True)
    pinned = [torch.empty(a.shape, dtype=torch.float32, pin_memory=True) for a in new]
    for p, a in zip(pinned, new):
        p.copy_(torch.from_numpy(a))
    ctx.set_cluster_params(aid, 1, *pinned)
    torch.cuda.synchronize()
    for got, want in zip(_stored(ctx, aid), new):
        assert np.array_equal(got, want)


@pytest.mark.parametrize("which", [0, 1, 2])
@pytest.mark.parametrize("shift", [0, 4])
def test_an_array_past_its_allocation_is_refused(hip, level, which, shift):
    ctx, aid, new, raw = level
    print(f"case: array {which} ends 4 bytes behind its allocation, {shift} bytes into it", flush=True)
    args = [None, None, None]
    args[which] = _At(raw.take(new[which].nbytes + shift - 4) + shift)
    with pytest.raises(hip.HairError) as e:
        ctx.set_cluster_params(aid, 1, *args)
    assert e.value.code == hip.HAIR_EDEVICE
