"""Device buffers that the kernels read and write themselves, and those that go through a copy
because they are not aligned to 16 bytes: the same numbers as through host arrays, bit for bit,
and nothing written beside the output."""
import numpy as np
import pytest

from paper_1204_2088_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hsf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1204_2088_amd import hsf as H
    H.load()
    return H


def slot(n, off, fill=None):
    """A device view of n doubles, off doubles from a 256-byte boundary, and its whole buffer."""
    import torch
    buf = torch.full((n + 4,), 7.0, dtype=torch.float64, device="cuda")
    v = buf[off:off + n]
    if fill is not None:
        v.copy_(torch.from_numpy(np.ascontiguousarray(fill).ravel()))
    return v, buf


def check(v, buf, off, ref):
    got = v.cpu().numpy()
    assert np.array_equal(got, np.asarray(ref).ravel())
    rest = buf.cpu().numpy()
    assert np.all(rest[:off] == 7.0) and np.all(rest[off + got.size:] == 7.0)


@pytest.mark.parametrize("off", [0, 1, 2])
# resident; a captured sequence; just below and above the size of direct launches
@pytest.mark.parametrize("L", [(16, 15, 12), (24, 20, 18), (40, 40, 40), (42, 40, 40)])
def test_device_buffers(hsf, L, off):
    import torch
    wl = W.Workload("place", L, W.chain(3, 4), True, W.chi_matrix(ab=15 / 7, bs=10 / 7), tau=1.0, noise=0.02, seed=3,
                    phi_p=0.3, precision="fp32")
    T = int(np.prod(L))
    rng = np.random.Generator(np.random.PCG64(2))
    w = 0.3 * rng.standard_normal((3,) + wl.shape)
    phi = W.initial_composition(wl)
    res = []
    for dev in (False, True):
        ctx = hsf.Context(wl, stream=torch.cuda.current_stream())
        ctx.set_densities(phi)
        ctx.set_fields(w)
        if not dev:
            out, q = ctx.evaluate()
            mu, f = ctx.mu_force()
            u = 1e-3 * rng.standard_normal(3 * T)
            ctx.cd_advance(mu, u)
            ctx.lb_advance(2, f)
            res = [np.array(v) for v in (out, q, mu, f, u, ctx.get_densities(), ctx.get_flow()[1])]
        else:
            (o, ob), (m, mb), (g, gb) = slot(3 * T, off), slot(3 * T, off), slot(3 * T, off)
            _, q = ctx.evaluate(out=o)
            check(o, ob, off, res[0])
            assert np.array_equal(q, res[1])
            ctx.mu_force(m, g)
            check(m, mb, off, res[2])
            check(g, gb, off, res[3])
            u, _ = slot(3 * T, off, res[4])
            ctx.cd_advance(m, u)
            ctx.lb_advance(2, g)
            assert np.array_equal(np.asarray(ctx.get_densities()).ravel(), res[5].ravel())
            assert np.array_equal(np.asarray(ctx.get_flow()[1]).ravel(), res[6].ravel())
        ctx.close()


@pytest.mark.parametrize("shift", [0, 2, 1, 5000, 25600 - 2, 25600, -2, -1, -25600])
def test_shared_outputs(hsf, shift):
    """Potential and force into overlapping device memory (force `shift` doubles after the
    potential): the force is the one of separate buffers and lies over the potential."""
    import torch
    wl = W.Workload("share", (32, 20, 20), W.chain(3, 4), False, W.chi_matrix(ab=15 / 7), tau=1.0, noise=0.2, seed=3)
    ctx = hsf.Context(wl, stream=torch.cuda.current_stream())
    ctx.set_densities(W.initial_composition(wl))
    ctx.set_fields(0.3 * np.random.default_rng(2).standard_normal((2,) + wl.shape))
    mu, f = ctx.mu_force()
    n, m = mu.size, f.size
    o = max(0, -shift)
    buf = torch.zeros(o + n + m + abs(shift), dtype=torch.float64, device="cuda")
    ctx.mu_force(buf[o:o + n], buf[o + shift:o + shift + m])
    want = np.zeros(buf.numel())
    want[o:o + n] = mu
    want[o + shift:o + shift + m] = f
    assert np.array_equal(buf.cpu().numpy(), want)
    ctx.close()


class Raw:
    """A device allocation of exactly `nbytes`, outside of torch's caching allocator, with the views
    the C interface takes."""

    def __init__(self, nbytes):
        import ctypes
        self.hip = ctypes.CDLL("libamdhip64.so.7")   # the runtime the library has loaded
        self.hip.hipMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t]
        self.hip.hipFree.argtypes = [ctypes.c_void_p]
        self.hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
        p = ctypes.c_void_p()
        assert self.hip.hipMalloc(ctypes.byref(p), nbytes) == 0
        self.p = p.value

    def put(self, a, at=0):
        a = np.ascontiguousarray(a)
        assert self.hip.hipMemcpy(self.p + at, a.ctypes.data, a.nbytes, 1) == 0

    def get(self, n, at=0):
        a = np.empty(n)
        assert self.hip.hipMemcpy(a.ctypes.data, self.p + at, a.nbytes, 2) == 0
        return a

    def free(self):
        self.hip.hipFree(self.p)


@pytest.mark.parametrize("spare", [0, 16, -16])
def test_ends_of_allocations(hsf, spare):
    """Buffers that end with their allocation (also from an offset into it) are taken; buffers whose
    allocation ends 16 bytes too early are refused by every call, as a copy refuses them.  The
    sizes are whole 4 KiB pages, so those 16 bytes are mapped memory all the same."""
    wl = W.Workload("ends", (8, 8, 8), W.chain(3, 4), False, W.chi_matrix(ab=15 / 7), tau=1.0, noise=0.2, seed=3)
    n, m = 2 * 512, 3 * 512
    rng = np.random.default_rng(4)
    phi, w = W.initial_composition(wl).ravel(), 0.3 * rng.standard_normal(n)
    u = 1e-3 * rng.standard_normal(m)
    ctx = hsf.Context(wl)
    ctx.set_densities(phi)
    ctx.set_fields(w)
    out, _ = ctx.evaluate()
    mu, f = ctx.mu_force()
    ctx.lb_advance(2, f)
    flow = ctx.get_flow()[1]
    ctx.cd_advance(mu, u)
    new = ctx.get_densities()
    ctx.close()
    ctx = hsf.Context(wl)
    ctx.set_densities(phi)
    ctx.set_fields(w)
    at = max(spare, 0)
    a, b, v = Raw(8 * n + spare), Raw(8 * m + spare), Raw(8 * m + spare)
    lib, h = ctx._lib, ctx._h
    if spare < 0:
        full = Raw(8 * m)
        assert lib.hsf_evaluate(h, a.p, None, hsf.DEVICE) == hsf.HSF_EHIP
        assert lib.hsf_mu_force(h, a.p, full.p, hsf.DEVICE) == hsf.HSF_EHIP
        assert lib.hsf_mu_force(h, full.p, b.p, hsf.DEVICE) == hsf.HSF_EHIP
        assert lib.hsf_lb_advance(h, 1, b.p, hsf.DEVICE) == hsf.HSF_EHIP
        assert lib.hsf_cd_advance(h, a.p, None, hsf.DEVICE) == hsf.HSF_EHIP
        assert lib.hsf_cd_advance(h, full.p, b.p, hsf.DEVICE) == hsf.HSF_EHIP
        assert np.array_equal(ctx.get_densities(), phi)
        full.hip.hipGetLastError()   # the runtime keeps the copies' error until it is read
        full.free()
    else:
        assert lib.hsf_evaluate(h, a.p + at, None, hsf.DEVICE) == hsf.HSF_OK
        assert np.array_equal(a.get(n, at), out)
        assert lib.hsf_mu_force(h, a.p + at, b.p + at, hsf.DEVICE) == hsf.HSF_OK
        assert np.array_equal(a.get(n, at), mu) and np.array_equal(b.get(m, at), f)
        assert lib.hsf_lb_advance(h, 2, b.p + at, hsf.DEVICE) == hsf.HSF_OK
        assert np.array_equal(ctx.get_flow()[1], flow)
        v.put(u, at)
        assert lib.hsf_cd_advance(h, a.p + at, v.p + at, hsf.DEVICE) == hsf.HSF_OK
        assert np.array_equal(ctx.get_densities(), new)
    ctx.close()
    for r in (a, b, v):
        r.free()


@pytest.mark.parametrize("tile,beads", [((64, 4, 4, -4), 8), ((64, 4, 4, -2), 40), ((32, 8, 2, -1), 2), ((32, 8, 2, -1), 12),
                                        ((32, 8, 2, 0), 2), ((8, 8, 8, 4), 3), ((8, 8, 8, 4), 40)])
def test_routes_of_an_evaluation(hsf, tile, beads):
    """Launches one by one into the caller's buffer, and a replayed sequence with a copy: which one an
    aligned buffer gets depends on the number of launches, a misaligned one always gets the
    copy; both give the bits of a host array."""
    import torch
    wl = W.Workload("routes", (44, 40, 40), W.chain(1, beads - 1), True, W.chi_matrix(ab=15 / beads, bs=10 / beads), tau=1.0,
                    noise=0.02, seed=3, phi_p=0.3, precision="fp32")
    ctx = hsf.Context(wl, stream=torch.cuda.current_stream())
    ctx.set_tile(tile)
    ctx.set_densities(W.initial_composition(wl))
    ctx.set_fields(0.3 * np.random.default_rng(2).standard_normal((3,) + wl.shape))
    ctx.evaluate()
    ref, q = ctx.evaluate()
    ref = ref.copy()
    for off in (0, 1, 0):
        v, buf = slot(3 * wl.V, off)
        assert np.array_equal(ctx.evaluate(out=v)[1], q)
        check(v, buf, off, ref)
    ctx.close()
