"""The row-resident paired sweeps (tilings with k <= -2: several contour steps of both sweeps
per launch) against the one-step kernels and the FP64 oracle.

Every stored value is the same expression of the same operands as in the one-step sequence;
only Q's sum over workgroups has another order.  A sum of at most about 100 additions per
level of its tree in FP64 differs by less than 2 * 100 * 2^-53 = 2.3e-14 relative, so densities
and Q agree with the one-step kernels of the same precision to 5e-14, in FP32 contexts too.
"""
import numpy as np
import pytest

from paper_1204_2088_amd import workloads as W

pytestmark = pytest.mark.gpu

ROWS = [(64, 4, 4, -2), (64, 4, 4, -4), (64, 8, 4, -2), (64, 8, 4, -3), (64, 8, 8, -2), (64, 8, 8, -3),
        (64, 8, 8, -4), (128, 8, 4, -2), (128, 8, 8, -3)]
SAME = 5e-14


@pytest.fixture(scope="module")
def hsf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1204_2088_amd import hsf as H
    H.load()
    return H


def workload(L, types, precision, solvent=False, seed=3):
    N = len(types)
    return W.Workload("rows", L, types, solvent, W.chi_matrix(ab=15 / N, bs=10 / N if solvent else 0.0), tau=1.0,
                      noise=0.02 if solvent else 0.2, seed=seed, phi_p=0.3 if solvent else 1.0, precision=precision)


def fields(wl, seed):
    return W.random_fields((wl.nsp,) + wl.shape, seed=seed, amplitude=1.2, smooth=1)


def rel(a, b):
    return np.max(np.abs(a - b)) / np.max(np.abs(b))


# whole 64- and 128-site rows, pieces of several widths, boxes smaller than tile and halo, odd
# and even numbers of step blocks, chains shorter than a block, single-bead species, solvent
CASES = [((64, 9, 7), W.chain(4, 4), False), ((128, 10, 6), W.chain(3, 9), True), ((17, 18, 20), W.chain(3, 4), False),
         ((130, 5, 9), W.chain(1, 3), False), ((61, 8, 8), W.chain(5, 11), False), ((59, 3, 1), W.chain(2, 3), False),
         ((1, 1, 2), W.chain(1, 1), False), ((5, 2, 3), W.chain(1, 2), True), ((128, 1, 17), W.chain(2, 4), False),
         ((33, 16, 12), W.chain(8, 8), False), ((64, 12, 13), W.chain(1, 0), False)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("L,types,solvent", CASES)
def test_rows_match_one_step(hsf, orc, precision, L, types, solvent):
    wl = workload(L, types, precision, solvent)
    w, phi = fields(wl, 5), W.initial_composition(wl)
    ctx = hsf.Context(wl)
    ctx.set_densities(phi.ravel())
    ctx.set_fields(w.ravel())
    ctx.set_tile((32, 8, 2, 0))
    ctx.evaluate()              # the FP32 scales follow the evaluation before
    one, q1 = ctx.evaluate()
    sysw = orc.System(L=wl.L, types=wl.types, has_solvent=wl.has_solvent, a=wl.a, chi=wl.chi, kappa=wl.kappa, dt=wl.dt,
                      tau=wl.tau)
    ref, qref = orc.evaluate(sysw, w, phi[:2].sum(0).mean(), phi[2].mean() if solvent else 0.0)
    tol = 1e-10 if precision == "fp64" else 1e-5
    ran = 0
    for t in ROWS:
        try:
            ctx.set_tile(t)
        except hsf.HsfError:    # 128-site rows on other boxes; bundles without an FP64 form
            assert (t[0] == 128 and L[0] != 128) or precision == "fp64", (t, L)
            continue
        two, q2 = ctx.evaluate()
        ran += 1
        print(f"[rows {t}] {L} N={len(types)} {precision}: {rel(two, one):.2e} from one step", flush=True)
        assert rel(two, one) <= SAME and abs(q2[0] / q1[0] - 1) <= SAME, (t, L)
        assert rel(two, ref.ravel()) < tol and abs(q2[0] / qref - 1) < tol, (t, L)
    assert ran >= 5, ran
    ctx.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("boxes", [[(64, 9, 7), (17, 18, 20)], [(17, 18, 20), (5, 3, 9), (64, 8, 8), (9, 7, 5), (70, 6, 11), (8, 8, 8)]])
def test_rows_batched_and_inverted(hsf, precision, boxes):
    """Uneven replicas in one context (descriptors as kernel arguments, and in device tables):
    evaluations as above, and the fields of an inversion (every replica its own line search)."""
    types = W.chain(3, 4)
    wls = [workload(L, types, precision, seed=r) for r, L in enumerate(boxes)]
    phi = np.concatenate([W.initial_composition(wl).ravel() for wl in wls])
    w = np.concatenate([fields(wl, 30 + r).ravel() for r, wl in enumerate(wls)])
    tol = 1e-9 if precision == "fp64" else 1e-4
    out = {}
    for t in [(32, 8, 2, 0)] + ROWS:
        ctx = hsf.Context(wls)
        try:
            ctx.set_tile(t)
        except hsf.HsfError:
            ctx.close()
            continue
        ctx.set_densities(phi)
        ctx.set_fields(w)
        ctx.evaluate()
        got, q = ctx.evaluate()
        ctx.set_fields(0.1 * w)
        ctx.invert(tol=tol, max_iter=500)
        res, _ = ctx.evaluate()
        out[t] = (got, q, res)
        ctx.close()
    one, q1, res1 = out.pop((32, 8, 2, 0))
    assert len(out) >= 5, list(out)
    for t, (got, q, res) in out.items():
        assert rel(got, one) <= SAME and np.max(np.abs(q / q1 - 1)) <= SAME, t
        assert np.max(np.abs(res - phi)) / np.max(np.abs(phi)) < 10 * tol, t


def test_rows_refined_inversion(hsf):
    """FP32 context whose bundle has no FP64 form: the FP64 phase takes its own, also when the
    flag is set after the tiling, and after a checkpoint."""
    wl = workload((64, 16, 16), W.chain(3, 5), "fp32")
    phi = W.initial_composition(wl)
    ctx = hsf.Context(wl)
    ctx.set_tile((64, 8, 8, -3))
    ctx.set_solver(refine=True)
    ctx.set_densities(phi.ravel())
    st, _ = ctx.invert(tol=1e-10, max_iter=2000, warm=hsf.WARM_LOCAL)
    assert st[0]["converged"] and st[0]["residual"] <= 1e-10
    ctx2 = hsf.Context(wl)
    ctx2.set_solver(refine=True)
    ctx2.set_state(ctx.get_state())
    assert ctx2.get_tile() == (64, 8, 8, -3)
    ctx.step(2, tol=1e-9)
    ctx2.step(2, tol=1e-9)
    assert np.array_equal(ctx.get_densities(), ctx2.get_densities())
    ctx.close()
    ctx2.close()


@pytest.mark.parametrize("precision,tile", [("fp64", (128, 8, 4, -2)), ("fp32", (128, 8, 4, -2)), ("fp32", (128, 8, 8, -3))])
def test_rows_repeat_bitwise(hsf, precision, tile):
    """The same evaluation 60 times over gives the same bits (a store whose data registers are
    overwritten too early shows in about one of ten evaluations of the FP64 bundle)."""
    wl = workload((128, 10, 6), W.chain(3, 9), precision, True)
    ctx = hsf.Context(wl)
    ctx.set_tile(tile)
    ctx.set_densities(W.initial_composition(wl).ravel())
    ctx.set_fields(fields(wl, 5).ravel())
    ctx.evaluate()
    ref, q = ctx.evaluate()
    for k in range(60):
        got, qk = ctx.evaluate()
        assert np.array_equal(got, ref) and np.array_equal(q, qk), k
    ctx.close()


@pytest.mark.parametrize("L,n,precision", [((64, 64, 64), 27, "fp64"), ((64, 64, 64), 25, "fp64"),
                                           ((41, 40, 40), 16, "fp32"), ((9, 7, 5), 2, "fp32"), ((9, 7, 5), 1, "fp64")])
def test_static_evaluation_at_its_limits(hsf, L, n, precision):
    """The allocation-free evaluation: the largest chains its array holds with one-step sweeps
    only (64^3, N = 27 in FP64) and with row sweeps (N = 25), both row bundles, the shortest
    chains; the same densities as hsf_evaluate (1e-10 relative, FP32 1e-5)."""
    import torch
    wl = workload(L, W.chain(n // 2, n - n // 2), precision)
    phi, w = W.initial_composition(wl) if n > 1 else np.ones((2,) + wl.shape) * [[[[0.0]]], [[[1.0]]]], fields(wl, 12)
    ctx = hsf.Context(wl)
    ctx.set_densities(phi.ravel())
    ctx.set_fields(w.ravel())
    ref, q = ctx.evaluate()
    ctx.close()
    wd, pd = torch.from_numpy(w.ravel().copy()).cuda(), torch.from_numpy(phi.ravel().copy()).cuda()
    out, qd = torch.zeros_like(wd), torch.zeros(1, dtype=torch.float64, device="cuda")
    assert hsf.evaluate_static(wl, wd, pd, out, qd) == hsf.HSF_OK
    torch.cuda.synchronize()
    tol = 1e-10 if precision == "fp64" else 1e-5
    assert rel(out.cpu().numpy(), ref) < tol and abs(qd.item() / q[0] - 1) < tol


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("L,n", [((1, 256, 40), 8), ((1, 90, 90), 8), ((6, 100, 100), 2), ((64, 64, 1), 2), ((1, 1, 4000), 12),
                                 ((3, 1, 700), 3)])
def test_static_evaluation_of_thin_boxes(hsf, orc, precision, L, n):
    """Boxes on both sides of the line between row sweeps and one-step sweeps (few sites per row, few
    rows), with a solvent, against the oracle."""
    import torch
    wl = workload(L, W.chain(1, n - 1), precision, True)
    phi, w = W.initial_composition(wl), fields(wl, 12)
    sysw = orc.System(L=wl.L, types=wl.types, has_solvent=True, a=wl.a, chi=wl.chi, kappa=wl.kappa, dt=wl.dt, tau=wl.tau)
    ref, qref = orc.evaluate(sysw, w, phi[:2].sum(0).mean(), phi[2].mean())
    wd, pd = torch.from_numpy(w.ravel().copy()).cuda(), torch.from_numpy(phi.ravel().copy()).cuda()
    out, qd = torch.zeros_like(wd), torch.zeros(1, dtype=torch.float64, device="cuda")
    for _ in range(2):
        assert hsf.evaluate_static(wl, wd, pd, out, qd) == hsf.HSF_OK
        torch.cuda.synchronize()
        tol = 1e-10 if precision == "fp64" else 1e-5
        assert rel(out.cpu().numpy(), ref.ravel()) < tol and abs(qd.item() / qref - 1) < tol
