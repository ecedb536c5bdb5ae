"""The column kernels of the chemical potential and the convection-diffusion update against
the FP64 oracle where their tilings can go wrong: whole rows of 64 and 128 sites, pieces of
one and several per row (62 sites at most), boxes thinner than a block's rows and planes,
uneven replicas (two sites per lane only when every row has 128), host and device buffers.

Bounds: mu sums about 60 terms below 10 in magnitude, 60 * 10 * 2^-53 < 1e-13; the update adds
six fluxes below 0.1 to values below 1, under 1e-15; the force is mu's gradient times
dt^2 phi < 1e-4, under 1e-15.
"""
import numpy as np
import pytest

from paper_1204_2088_amd import workloads as W

pytestmark = pytest.mark.gpu

BOXES = [(64, 5, 6), (128, 4, 7), (62, 3, 4), (63, 9, 2), (130, 2, 5), (125, 6, 3), (17, 18, 20), (5, 3, 9), (1, 1, 2),
         (2, 1, 1), (128, 1, 1)]


@pytest.fixture(scope="module")
def hsf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1204_2088_amd import hsf as H
    H.load()
    return H


def workload(L, solvent, seed=1):
    types = W.chain(3, 5)
    return W.Workload("columns", L, types, solvent, W.chi_matrix(ab=20 / 8, bs=10 / 8 if solvent else 0.0), tau=1.0,
                      noise=0.05, seed=seed, phi_p=0.4 if solvent else 1.0)


def system(orc, wl, **kw):
    return orc.System(L=wl.L, types=wl.types, has_solvent=wl.has_solvent, a=wl.a, chi=wl.chi, kappa=wl.kappa, dt=wl.dt,
                      tau=wl.tau, **kw)


def inputs(wl, seed):
    rng = np.random.default_rng(seed)
    phi = rng.uniform(0.1, 0.5, (wl.nsp,) + wl.shape)
    return phi, rng.standard_normal(phi.shape), 0.05 * rng.standard_normal((3,) + wl.shape)


def check(orc, wl, phi, w, u, mu, f, new, new0, **kw):
    s = system(orc, wl, **kw)
    mu_ref, f_ref = orc.mu_force(s, phi, w)
    assert np.max(np.abs(mu.reshape(phi.shape) - mu_ref)) < 1e-13
    assert np.max(np.abs(f.reshape(u.shape) - f_ref)) < 1e-15
    assert np.max(np.abs(new.reshape(phi.shape) - orc.cd_update(s, phi, mu_ref, u))) < 1e-15
    assert np.max(np.abs(new0.reshape(phi.shape) - orc.cd_update(s, phi, mu_ref))) < 1e-15


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("solvent", [False, True])
@pytest.mark.parametrize("boxes", [[b] for b in BOXES] + [[(128, 3, 4), (128, 5, 2)], [(128, 3, 4), (64, 6, 5), (7, 6, 5)]])
def test_columns_match_oracle(hsf, orc, boxes, solvent, device):
    import torch
    wls = [workload(L, solvent, r) for r, L in enumerate(boxes)]
    data = [inputs(wl, 7 + r) for r, wl in enumerate(wls)]
    cat = lambda k: np.concatenate([d[k].ravel() for d in data])
    put = (lambda a: torch.from_numpy(a).cuda()) if device else (lambda a: a)
    new = (lambda n: torch.zeros(n, dtype=torch.float64, device="cuda")) if device else (lambda n: np.zeros(n))
    get = lambda a: a.cpu().numpy() if device else a
    ctx = hsf.Context(wls)
    ctx.set_densities(put(cat(0)))
    ctx.set_fields(put(cat(1)))
    mu, f = ctx.mu_force(new(ctx.nsp * ctx.T), new(3 * ctx.T))
    ctx.cd_advance(mu, put(cat(2)))
    out = ctx.get_densities()
    ctx.set_densities(put(cat(0)))
    ctx.cd_advance(mu)
    out0 = ctx.get_densities()
    mu, f = get(mu), get(f)
    for r, wl in enumerate(wls):
        a, b = ctx.field_offset(r), ctx.site_offset(r)
        n, V = wl.nsp * wl.V, wl.V
        check(orc, wl, *data[r], mu[a:a + n], f[3 * b:3 * b + 3 * V], out[a:a + n], out0[a:a + n])
    ctx.close()


@pytest.mark.parametrize("L", [(64, 3, 4), (128, 2, 3), (63, 5, 2), (9, 7, 5)])
def test_columns_with_noise(hsf, orc, L):
    wl = workload(L, True)
    phi, mu, u = inputs(wl, 3)
    ctx = hsf.Context(wl)
    ctx.set_noise(cd=True, lb=False, omega=400.0, seed=11, step=5)
    ctx.set_densities(phi.ravel())
    ctx.cd_advance(mu.ravel(), u.ravel())
    ref = orc.cd_update(system(orc, wl, noise=1, omega=400.0, seed=11, step=5), phi, mu, u)
    assert np.max(np.abs(ctx.get_densities().reshape(phi.shape) - ref)) < 1e-15
    ctx.close()


def test_update_then_evaluate(hsf):
    """The updated densities are the current ones for the calls that follow (captured
    sequences of both density buffers), as when they are read back and set."""
    wl = workload((20, 18, 16), False).with_(precision="fp32")
    phi, mu, u = inputs(wl, 4)
    phi[1] = 1.0 - phi[0]
    ctx, ctx2 = hsf.Context(wl), hsf.Context(wl)
    w = W.random_fields(phi.shape, seed=2, amplitude=0.5, smooth=1)
    ctx.set_fields(w.ravel())
    ctx.set_densities(phi.ravel())
    for k in range(4):
        ctx.cd_advance(0.01 * mu.ravel(), 0.01 * u.ravel())
        cur = ctx.get_densities()
        ctx2.set_fields(w.ravel())
        ctx2.set_densities(cur)
        a, qa = ctx.evaluate()
        b, qb = ctx2.evaluate()
        assert np.array_equal(a, b) and np.array_equal(qa, qb), k
    ctx.close()
    ctx2.close()


# rows that share a wavefront: one site to thirty, numbers of rows that do not fill the last
# group or the block, batches where most sites (not all rows) are short
SHORT = [[(1, 17, 5)], [(1, 90, 3)], [(2, 9, 4)], [(3, 53, 2)], [(4, 23, 6)], [(10, 33, 3)], [(16, 20, 9)], [(29, 9, 5)],
         [(30, 8, 4)], [(31, 7, 4)], [(4, 30, 5), (9, 7, 6)], [(6, 40, 4), (70, 3, 4)], [(128, 3, 2), (8, 40, 6)],
         [(64, 5, 2), (20, 40, 3), (1, 1, 1)]]


@pytest.mark.parametrize("noise", [False, True])
@pytest.mark.parametrize("solvent", [False, True])
@pytest.mark.parametrize("boxes", SHORT)
def test_short_rows_match_oracle(hsf, orc, boxes, solvent, noise):
    wls = [workload(L, solvent, r) for r, L in enumerate(boxes)]
    data = [inputs(wl, 17 + r) for r, wl in enumerate(wls)]
    cat = lambda k: np.concatenate([d[k].ravel() for d in data])
    ctx = hsf.Context(wls)
    ctx.set_densities(cat(0))
    ctx.set_fields(cat(1))
    mu, f = ctx.mu_force()
    if noise:
        ctx.set_noise(cd=True, lb=False, omega=400.0, seed=11, step=5)
    ctx.cd_advance(mu, cat(2))
    out = ctx.get_densities()
    ctx.set_densities(cat(0))
    if noise:
        ctx.set_noise(cd=True, lb=False, omega=400.0, seed=11, step=5)
    ctx.cd_advance(mu)
    out0 = ctx.get_densities()
    for r, wl in enumerate(wls):
        a, b = ctx.field_offset(r), ctx.site_offset(r)
        n, V = wl.nsp * wl.V, wl.V
        kw = dict(noise=1, omega=400.0, seed=11, rep=r, step=5) if noise else {}
        check(orc, wl, *data[r], mu[a:a + n], f[3 * b:3 * b + 3 * V], out[a:a + n], out0[a:a + n], **kw)
    ctx.close()
