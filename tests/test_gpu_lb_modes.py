"""The LB step's variants (BGK, MRT, a batch that mixes them; with and without mode noise) over
several steps of one call, with the density and velocity of the last, against the FP64 oracle.

Tolerance: populations of size 1/36 to 1/3, about 100 additions each over the transforms and the
steps: 100 * 2^-53 * 1/3 < 4e-15; 1e-14 leaves a factor for the noise's square roots, and
3e-14 on the sum of 19 of them.
"""
import numpy as np
import pytest

from paper_1204_2088_amd import workloads as W

pytestmark = pytest.mark.gpu

OMEGA = 300.0


@pytest.fixture(scope="module")
def hsf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1204_2088_amd import hsf as H
    H.load()
    return H


def system(orc, wl, **kw):
    s = orc.System(L=wl.L, types=wl.types, has_solvent=wl.has_solvent, a=wl.a, chi=wl.chi, kappa=wl.kappa, dt=wl.dt,
                   tau=wl.tau, hydro=wl.hydro)
    if wl.lb == "mrt":
        s.lb_mode = 1
        s.gamma_s, s.gamma_b, s.gamma_ghost = wl.gammas
    for k, v in kw.items():
        setattr(s, k, v)
    return s


def melt(L, tau):
    return W.Workload("lb_modes", L, W.chain(2, 2), False, W.chi_matrix(ab=5.0), tau=tau, noise=0.01, seed=1,
                      precision="fp64")


@pytest.mark.parametrize("noise", [False, True])
@pytest.mark.parametrize("modes", [("bgk",), ("mrt",), ("mrt", "bgk"), ("bgk", "mrt", "mrt")])
def test_modes(hsf, orc, modes, noise):
    boxes = [(9, 7, 11), (16, 5, 6), (3, 20, 4)]
    wls = [melt(L, 0.8 + 0.2 * k).with_(lb=m, gammas=(0.3, -0.2, 0.1)) for k, (L, m) in enumerate(zip(boxes, modes))]
    rng = np.random.default_rng(8)
    ns = [np.ascontiguousarray(orc.lb_rest_state(system(orc, w)) * (1 + 0.03 * rng.uniform(-1, 1, (19,) + w.shape)))
          for w in wls]
    fs = [np.ascontiguousarray(2e-3 * rng.uniform(-1, 1, (3,) + w.shape)) for w in wls]
    ctx = hsf.Context(wls)
    if noise:
        ctx.set_noise(cd=False, lb=True, omega=OMEGA, seed=6, step=4)
    ctx.set_lb(np.concatenate([n.ravel() for n in ns]))
    ctx.lb_advance(3, np.concatenate([f.ravel() for f in fs]))
    got = ctx.get_lb()
    rho, u = ctx.get_flow()
    ctx.close()
    o = 0
    for r, wl in enumerate(wls):
        ref = ns[r]
        for k in range(3):
            kw = dict(noise=2, omega=OMEGA, seed=6, rep=r, step=4 + k) if noise else {}
            ref, rref, uref = orc.lb_step(system(orc, wl, **kw), ref, fs[r])
        V = int(np.prod(wl.L))
        assert np.max(np.abs(got[19 * o:19 * (o + V)] - ref.ravel())) < 1e-14
        assert np.max(np.abs(rho[o:o + V] - rref.ravel())) < 3e-14
        assert np.max(np.abs(u[3 * o:3 * (o + V)] - uref.ravel())) < 3e-14
        o += V
