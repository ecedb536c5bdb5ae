"""Evaluations and inversions of small boxes in one workgroup per replica, the default there,
against the one-step kernels (an explicit tiling) and the FP64 oracle.

The two paths store the same expressions of the same operands (in FP64 with rows of 16 sites up to
the order of four additions, a few 2^-53 per step); sums over sites differ in order only (at most 4096 terms in trees about 100 deep: 2 * 100 * 2^-53 < 5e-14 relative on Q and
the densities, in FP32 contexts too).
"""
import numpy as np
import pytest

from paper_1204_2088_amd import workloads as W

pytestmark = pytest.mark.gpu

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
    return W.Workload("resident", L, types, solvent, W.chi_matrix(ab=15 / N, bs=10 / N if solvent else 0.0), tau=1.0,
                      noise=0.02 if solvent else 0.2, seed=seed, phi_p=0.3 if solvent else 1.0, precision=precision)


def fields(wl, seed, amp=1.0):
    return W.random_fields((wl.nsp,) + wl.shape, seed=seed, amplitude=amp, smooth=1)


def rel(a, b):
    return np.max(np.abs(a - b)) / np.max(np.abs(b))


# the largest box, rows and planes that do not fill the layout, one to four planes in the last
# column, boxes that wrap onto themselves, single-bead species, the longest chain
CASES = [((16, 16, 16), W.chain(4, 4), False), ((16, 16, 16), W.chain(3, 9), True), ((16, 15, 13), W.chain(3, 4), False),
         ((15, 16, 4), W.chain(2, 3), False), ((5, 3, 9), W.chain(2, 3), True), ((1, 1, 2), W.chain(1, 1), False),
         ((3, 1, 1), W.chain(1, 0), False), ((12, 11, 10), W.chain(5, 59), False), ((13, 14, 15), W.chain(4, 4), False),
         ((7, 8, 8), W.chain(3, 5), False)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("L,types,solvent", CASES)
def test_resident_evaluation(hsf, orc, precision, L, types, solvent):
    wl = workload(L, types, precision, solvent)
    w = fields(wl, 5)
    phi = W.initial_composition(wl) if len(types) > 1 else np.stack([np.ones(wl.shape), np.zeros(wl.shape)])
    out = []
    for explicit in (False, True):
        ctx = hsf.Context(wl)
        if explicit:
            ctx.set_tile((32, 8, 2, 0))
        ctx.set_densities(phi.ravel())
        ctx.set_fields(w.ravel())
        ctx.evaluate()
        out.append(ctx.evaluate())
        out[-1] += (ctx.observables()[0],)
        ctx.close()
    (a, qa, fa), (b, qb, fb) = out
    sysw = orc.System(L=wl.L, types=wl.types, has_solvent=wl.has_solvent, a=wl.a, chi=wl.chi, kappa=wl.kappa, dt=wl.dt,
                      tau=wl.tau)
    ref, qref = orc.evaluate(sysw, w, phi[:2].sum(0).mean(), phi[2].mean() if solvent else 0.0)
    print(f"[resident] {L} N={len(types)} {precision}: {rel(a, b):.2e} from one step", flush=True)
    assert rel(a, b) <= SAME and abs(qa[0] / qb[0] - 1) <= SAME
    assert abs(fa[0] - fb[0]) < 1e-11 * (1 + abs(fb[0]))
    tol = 1e-10 if precision == "fp64" else 1e-5
    assert rel(a, ref.ravel()) < tol and abs(qa[0] / qref - 1) < tol


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("precond", [False, True])
def test_resident_inversion(hsf, precision, precond):
    """Uneven replicas, each with its own line search, plain and preconditioned, refined below
    1e-5 in FP32 contexts: the residual is reached, the fields are those of the one-step path
    (both are within the tolerance of the solution), the counts differ by rounding only, and a
    limit on the iterations stops both alike."""
    boxes = [(16, 16, 16), (9, 7, 5), (12, 6, 10)]
    wls = [workload(L, W.chain(3, 5), precision, True, seed=r) for r, L in enumerate(boxes)]
    phi = np.concatenate([W.initial_composition(wl).ravel() for wl in wls])
    out = []
    for explicit in (False, True):
        ctx = hsf.Context(wls)
        if explicit:
            ctx.set_tile((32, 8, 2, 0))
        ctx.set_solver(precond=precond, refine=True)
        ctx.set_densities(phi)
        st, _ = ctx.invert(tol=1e-9, max_iter=3000, warm=hsf.WARM_LOCAL)
        w = ctx.get_fields()
        new, _ = ctx.evaluate()
        ctx.set_fields(np.zeros_like(w))
        few, rc = ctx.invert(tol=1e-9, max_iter=3, allow_noconv=True)
        assert rc == hsf.HSF_ENOCONV and all(s["iterations"] in (3, 6) for s in few)
        out.append((st, w, new, few))
        ctx.close()
    (sa, wa, na, fa), (sb, wb, nb, fb) = out
    assert all(s["converged"] and s["residual"] <= 1e-9 for s in sa + sb)
    assert np.max(np.abs(wa - wb)) < 1e-6 * np.max(np.abs(wb))
    assert all(abs(a["iterations"] - b["iterations"]) <= 3 + 0.1 * b["iterations"] for a, b in zip(sa, sb))
    assert all(abs(a["residual"] / b["residual"] - 1) < 1e-3 for a, b in zip(fa, fb))


def test_resident_many_passes_and_nonfinite(hsf):
    """An inversion of more passes than one launch takes; a NaN field in one replica leaves the
    others' results as they are without it."""
    wls = [workload((8, 8, 8), W.chain(3, 5), "fp64", True, seed=r) for r in range(3)]
    phi = np.concatenate([W.initial_composition(wl).ravel() for wl in wls])
    ctx = hsf.Context(wls)
    ctx.set_densities(phi)
    st, _ = ctx.invert(tol=0.0, max_iter=200, warm=hsf.WARM_LOCAL, allow_noconv=True)
    assert max(s["evaluations"] for s in st) > 129
    w = ctx.get_fields()
    ref, q = ctx.evaluate()
    bad = w.copy()
    fo = ctx.field_offset(1)
    bad[fo + 5] = np.nan
    ctx.set_fields(bad)
    out = np.zeros_like(ref)
    with pytest.raises(hsf.HsfError) as e:
        ctx.evaluate(out)
    assert e.value.code == hsf.HSF_ENONFINITE
    n = 3 * wls[0].V
    assert np.array_equal(out[:n], ref[:n]) and np.array_equal(out[2 * n:], ref[2 * n:])
    ctx.close()


def test_resident_state_round_trip(hsf):
    """A run continued from a checkpoint repeats bit for bit, with the path it was written with."""
    wl = workload((12, 12, 12), W.chain(4, 4), "fp32")
    for tile in (None, (32, 8, 2, -1)):
        ctx = hsf.Context(wl)
        if tile:
            ctx.set_tile(tile)
        ctx.set_densities(W.initial_composition(wl).ravel())
        ctx.step(2, tol=1e-5)
        buf = ctx.get_state()
        ctx.step(3, tol=1e-5)
        ctx2 = hsf.Context(wl)
        ctx2.set_state(buf)
        ctx2.step(3, tol=1e-5)
        assert np.array_equal(ctx.get_densities(), ctx2.get_densities())
        assert np.array_equal(ctx.get_fields(), ctx2.get_fields())
        ctx.close()
        ctx2.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("L", [(16, 16, 16), (16, 15, 13), (13, 14, 16), (3, 1, 1)])
def test_resident_one_bead(hsf, orc, precision, L):
    """Chains of one bead, whose evaluation has no contour step after Q, on boxes that fill all
    wavefronts of the workgroup: the first evaluation of a fresh context and those after a change
    of the fields (every one has another Q), then the line searches of an inversion (a B amount
    that no bead makes keeps it from converging), against the oracle and the one-step kernels.
    The fields after four iterations differ by rounding, in FP32 contexts that of the propagators
    (2^-24 a site, in step lengths of order one)."""
    wl = workload(L, W.chain(1, 0), precision)
    sysw = orc.System(L=wl.L, types=wl.types, has_solvent=False, a=wl.a, chi=wl.chi, kappa=wl.kappa, dt=wl.dt, tau=wl.tau)
    rng = np.random.default_rng(2)
    tol = 1e-10 if precision == "fp64" else 1e-5
    phi = np.stack([0.8 + 0.1 * rng.random(wl.shape), np.full(wl.shape, 0.1)])
    inverted = []
    for tile in (None, (32, 8, 2, 0)):
        ctx = hsf.Context(wl)
        if tile:
            ctx.set_tile(tile)
        ctx.set_densities(phi.ravel())
        for k, shift in enumerate((0.0, 2.0, -1.5, 0.7, 3.0)):
            w = fields(wl, 5 + k) + shift
            ctx.set_fields(w.ravel())
            got, q = ctx.evaluate()
            ref, qref = orc.evaluate(sysw, w, phi.sum(0).mean(), 0.0)
            assert rel(got, ref.ravel()) < tol and abs(q[0] / qref - 1) < tol, (tile, k)
        ctx.set_fields(0.2 * fields(wl, 9).ravel())
        st, rc = ctx.invert(tol=1e-12, max_iter=4, allow_noconv=True)
        assert rc == hsf.HSF_ENOCONV and st[0]["iterations"] == 4
        inverted.append(ctx.get_fields())
        ctx.close()
    assert rel(*inverted) < (1e-10 if precision == "fp64" else 1e-5)


def runs_resident(ctx):
    """Whether evaluations take one workgroup per replica: a single launch, with no density
    launch after the sweeps."""
    ctx.set_timing(True)
    ctx.get_timing()
    ctx.evaluate()
    t = ctx.get_timing()
    ctx.set_timing(False)
    return t["bwd"][1] == 0 and t["pair"][1] > 0


def test_autotune_takes_the_faster_path(hsf):
    """One workgroup per replica at 16^3 (calls of 46 us against 68), launches for 1024 boxes of 16
    sites and 64 beads (485 against 718).  Nothing of autotune's own is left in the timing."""
    for boxes, types, resident in ([(16, 16, 16)], W.chain(4, 4), True), ([(16, 1, 1)] * 1024, W.chain(32, 32), False):
        wls = [workload(L, types, "fp64", seed=r) for r, L in enumerate(boxes)]
        ctx = hsf.Context(wls)
        assert runs_resident(ctx)          # the default of small boxes
        ctx.set_densities(np.concatenate([W.initial_composition(wl).ravel() for wl in wls]))
        ctx.set_timing(True)
        ctx.autotune(2)
        assert all(n == 0 for _, n in ctx.get_timing().values())
        assert runs_resident(ctx) == resident
        ctx.close()


def test_autotune_keeps_the_scales(hsf):
    """The per-step scales of an FP32 context are those of its evaluations, not of the timing runs:
    fields of 10 ln 2 give every step the exponent -10 (csum is 1), which a checkpoint holds as a run
    of N equal integers; other fields change nothing until they are evaluated."""
    wl = workload((12, 8, 8), W.chain(4, 4), "fp32")
    ctx = hsf.Context(wl)
    ctx.set_densities(W.initial_composition(wl).ravel())
    ctx.set_fields(np.full(2 * wl.V, 10 * np.log(2.0)))
    ctx.evaluate()

    def scales():
        n = ctx.get_state().size - 8 * (6 * 2 + 19) * wl.V   # header and replica states
        return ctx.get_state()[:n // 4 * 4].view(np.int32)

    run = lambda v, x: any(np.all(v[k:k + wl.N] == x) for k in range(v.size - wl.N))
    assert run(scales(), -10)
    ctx.set_fields(np.full(2 * wl.V, 3 * np.log(2.0)))
    ctx.autotune(2)
    assert run(scales(), -10)
    ctx.evaluate()
    assert run(scales(), -3) and not run(scales(), -10)
    ctx.close()


def test_state_version(hsf):
    """A checkpoint with resident evaluations carries version 2, which a library without them
    refuses, one with launches version 1 as ever; version 1 with the resident bit (bit 1 of the
    fields' word) is taken as well, other versions are refused."""
    wl = workload((12, 12, 12), W.chain(4, 4), "fp32")
    ctx = hsf.Context(wl)
    ctx.set_densities(W.initial_composition(wl).ravel())
    ctx.step(1, tol=1e-5)
    buf = ctx.get_state()
    version = lambda b: int(b[8:12].view(np.int32)[0])   # after the 64-bit magic
    assert version(buf) == 2
    ctx.set_tile((32, 8, 2, -1))
    assert version(ctx.get_state()) == 1 and not runs_resident(ctx)
    ctx.set_state(buf)
    assert runs_resident(ctx)
    for v, ok in ((1, True), (0, False), (3, False)):
        ctx.set_tile((32, 8, 2, -1))
        other = buf.copy()
        other[8:12] = np.frombuffer(np.int32(v).tobytes(), np.uint8)
        if ok:
            ctx.set_state(other)
            assert runs_resident(ctx)
        else:
            with pytest.raises(hsf.HsfError):
                ctx.set_state(other)
            assert not runs_resident(ctx)
    ctx.close()
