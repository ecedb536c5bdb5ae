"""Loss gradients of the network at the sizes where the weight-gradient kernel's tiles, slices and
channel octets have edges, against the FP64 oracle.

Tolerance: each layer on the way rounds its operands to bfloat16 (2^-9 relative each, data and
weights); over the at most 15 convolutions forward and 15 backward these add like independent
errors, 2^-9 sqrt(30 * 2) = 1.5e-2 at worst where no sum over sites averages them.  A
missing row, tile, slice or channel moves a layer's gradient by O(1).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 2e-2


@pytest.fixture(scope="module")
def hsf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1204_2088_amd import hsf as H
    H.load()
    return H


def smooth(rng, shape):
    x = rng.standard_normal(shape)
    for ax in (2, 3, 4):
        x = (np.roll(x, 1, ax) + x + np.roll(x, -1, ax)) / 3.0
    return (x / np.std(x)).astype(np.float32)


@pytest.mark.parametrize("B,L,in_ch,widths", [
    (5, 32, 2, (32,)),            # more tiles than slices, two output tiles, four octets
    (5, 64, 1, (8,)),             # the widest tile, more tiles than slices
    (1, 32, 3, (12, 20)),         # octets that are not full; every input composition
    (2, 20, 2, (8,)),             # the narrow tile pads x; rows in wide loads
    (1, 28, 2, (4, 9)),           # a level with L a multiple of 4 and one without
    (1, 4, 2, (16,)),             # boxes smaller than a tile
    (3, 5, 2, (8,)),
    (2, 1, 2, (8,)),
    (1, 8, 6, (8, 16, 24, 32)),   # down to one site
    (2, 24, 9, (17, 8, 31)),      # a coarser level narrower than the finer
])
def test_gradient_at_edges(hsf, B, L, in_ch, widths):
    from oracle import net_oracle as NO
    rng = np.random.Generator(np.random.PCG64(31))
    net = hsf.Net(in_ch, 2, widths, seed=4)
    p = net.get_params()
    p = (p + 0.05 * rng.standard_normal(p.size)).astype(np.float32)
    net.set_params(p)
    x, t = smooth(rng, (B, in_ch, L, L, L)) if L > 1 else rng.standard_normal((B, in_ch, 1, 1, 1)).astype(np.float32), \
        rng.standard_normal((B, 2, L, L, L)).astype(np.float32)
    loss, g = net.loss_grad(x.ravel(), t.ravel(), B, L)
    again = net.loss_grad(x.ravel(), t.ravel(), B, L)
    net.close()
    assert again[0] == loss and np.array_equal(again[1], g)
    lref, gref = NO.loss_and_grad(p, x, t, in_ch, 2, widths, bf16=True)
    gref = np.asarray(gref)
    assert abs(loss - lref) <= 1e-3 * lref
    off = 0
    for l, (ci, co) in enumerate(NO.layer_shapes(in_ch, 2, widths)):
        n = co * ci * 27
        for part in (slice(off, off + n), slice(off + n, off + n + co)):   # weights, bias
            a, b = g[part].astype(np.float64), gref[part]
            assert np.linalg.norm(a - b) <= TOL * np.linalg.norm(b), (l, part)
        off += n + co
