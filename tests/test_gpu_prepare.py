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
