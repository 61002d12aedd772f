"""The variance tables of the Myrtle kernels at the edges of their split: one
to four stages (coarse slices by part or whole), stages without layers, one
and several channels, and more images than one scratch pass holds."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_05420_amd import ops
    return ops


@pytest.mark.parametrize("hw,c,depth,sb2", [
    (2, 1, (1,), 0.01), (8, 3, (3,), 0.0), (4, 2, (1, 2), 0.01), (16, 4, (4, 1), 0.0), (16, 3, (2, 0, 1), 0.01),
    (16, 3, (1, 1, 1, 1), 0.0), (32, 1, (1, 0, 2, 1), 0.01), (32, 3, (2, 1, 1, 1), 0.0),
])
def test_tables_over_stage_counts(nk, hw, c, depth, sb2):
    """The kernel of every network shape against the float64 oracle, within
    the parity bar of float32 stages (2e-5 normalised)."""
    x1 = synth.iid_images(3, hw, hw, c, 11)
    x2 = synth.iid_images(4, hw, hw, c, 12)
    print(f"tables hw {hw} c {c} depth {depth}", flush=True)
    k = nk.myrtle_nngp(torch.from_numpy(x1).cuda(), torch.from_numpy(x2).cuda(), depth, 2.0, sb2).cpu().numpy()
    net = oracle.Myrtle(depth, 2.0, sb2)
    ref = oracle.myrtle_gram(x1, x2, net)
    d1, d2 = (np.sqrt(np.diag(oracle.myrtle_gram(x, None, net))) for x in (x1, x2))
    err = np.max(np.abs(k - ref) / np.outer(d1, d2))
    print(f"  normalised error {err:.2e}", flush=True)
    assert err <= 2e-5


@pytest.mark.parametrize("n1,n2", [(2050, 2), (3, 2046), (2048, 1)])
def test_tables_over_scratch_passes(nk, n1, n2):
    """Images on both sides of the 2048-image scratch pass, and a pass that
    ends inside the second set: the rows and columns there equal those of a
    block of their own, bit for bit."""
    x1 = torch.from_numpy(synth.iid_images(n1, 8, 8, 3, 21)).cuda()
    x2 = torch.from_numpy(synth.iid_images(n2, 8, 8, 3, 22)).cuda()
    print(f"tables {n1} + {n2} images", flush=True)
    k = nk.myrtle_nngp(x1, x2, (2, 1, 1), 2.0, 0.0)
    a, b = slice(max(0, n1 - 4), n1), slice(max(0, n2 - 4), n2)
    part = nk.myrtle_nngp(x1[a].contiguous(), x2[b].contiguous(), (2, 1, 1), 2.0, 0.0)
    assert torch.equal(k[a, b], part)


@pytest.mark.parametrize("hw,c,depth,sb2", [(8, 1, (2,), 0.02), (16, 2, (1, 2), 0.0), (16, 3, (2, 0, 1), 0.02),
                                            (16, 3, (1, 1, 1, 1), 0.0), (32, 1, (1, 0, 1, 1), 0.02)])
def test_self_adjoint_over_stage_counts(nk, hw, c, depth, sb2):
    """The adjoint of every network shape against the float64 autograd oracle,
    within the adjoint's bar (1e-5 of the largest entry)."""
    from oracle import grad as ograd

    x1 = synth.correlated_images(2, hw, hw, c, 3.0, 31)
    x2 = synth.correlated_images(1, hw, hw, c, 3.0, 32)
    g = np.array([[0.7], [-1.2]], dtype=np.float32)
    print(f"adjoint hw {hw} c {c} depth {depth}", flush=True)
    dx1, dx2, ds = nk.myrtle_nngp_backward(torch.from_numpy(x1).cuda(), torch.from_numpy(x2).cuda(),
                                           torch.from_numpy(g).cuda(), depth, 2.0, sb2)
    r1, r2, rs, _ = ograd.myrtle_vjp(x1, x2, np.array([[0, 0], [1, 0]]), g.ravel(), depth, 2.0, sb2)
    for got, want in ((dx1, r1), (dx2, r2), (ds, rs)):
        err = np.max(np.abs(got.cpu().numpy() - want)) / np.max(np.abs(want))
        print(f"  relative error {err:.2e}", flush=True)
        assert err <= 1e-5


@pytest.mark.parametrize("n1,n2", [(513, 1), (2, 511), (1, 512)])
def test_self_adjoint_over_scratch_passes(nk, n1, n2):
    """Images on both sides of the 512-image scratch pass: the gradients of the
    last images equal those of a block of their own.  Both are float64 sums
    (in no fixed order) rounded to float32: one rounding, 1.2e-7, apart at most."""
    x1 = torch.from_numpy(synth.iid_images(n1, 8, 8, 3, 41)).cuda()
    x2 = torch.from_numpy(synth.iid_images(n2, 8, 8, 3, 42)).cuda()
    a, b = max(0, n1 - 2), max(0, n2 - 2)
    g = torch.zeros((n1, n2), device="cuda")
    g[a:, b:] = torch.arange(1, (n1 - a) * (n2 - b) + 1, device="cuda").reshape(n1 - a, n2 - b)
    print(f"adjoint {n1} + {n2} images", flush=True)
    dx1, dx2, ds = nk.myrtle_nngp_backward(x1, x2, g, (2, 1, 1), 2.0, 0.0)
    e1, e2, es = nk.myrtle_nngp_backward(x1[a:].contiguous(), x2[b:].contiguous(), g[a:, b:].contiguous(), (2, 1, 1),
                                         2.0, 0.0)
    for got, want in ((dx1[a:], e1), (dx2[b:], e2), (ds, es)):
        assert torch.allclose(got, want, rtol=1.3e-7, atol=0.0)
    assert torch.count_nonzero(dx1[:a]) == 0 and torch.count_nonzero(dx2[:b]) == 0
