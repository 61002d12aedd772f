"""A 32x32 stage shares the sweep of a pair among workgroups when there are few
pairs.  The pooled rows are summed in the order of the whole sweep, so a block
of few pairs (from one pair, 16 parts, to 255, the last two-part size or none)
must equal, bit for bit, the same rows of a block too large to be split."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth,c,sb2", [((3, 3, 3), 3, 0.0), ((1, 1), 4, 0.01), ((2, 1, 1), 1, 0.01), ((3, 0, 1), 3, 0.0)])
def test_split_sweep_is_the_whole_sweep(depth, c, sb2):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_05420_amd import ops
    a = torch.from_numpy(synth.iid_images(40, 32, 32, c, 21)).cuda()
    b = torch.from_numpy(synth.iid_images(85, 32, 32, c, 22)).cuda()
    whole = ops.myrtle_nngp(a, b, depth, 2.0, sb2)
    assert bool(torch.isfinite(whole).all())
    for n1, n2 in ((1, 1), (1, 3), (2, 8), (3, 11), (2, 32), (2, 60), (3, 43), (2, 85), (3, 85)):
        print(f"depth {depth} {n1} x {n2}", flush=True)
        assert torch.equal(ops.myrtle_nngp(a[:n1].contiguous(), b[:n2].contiguous(), depth, 2.0, sb2), whole[:n1, :n2])
    sym = ops.myrtle_nngp(b, None, depth, 2.0, sb2)
    few = ops.myrtle_nngp(b[:9].contiguous(), None, depth, 2.0, sb2)
    assert torch.equal(few, sym[:9, :9])


@pytest.mark.parametrize("depth,c,sb2", [((2, 2, 2), 3, 0.0), ((1, 1), 4, 0.01)])
def test_split_sweep_of_64x64(depth, c, sb2):
    """The same of the 64x64 first stage, up to 32 parts."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_05420_amd import ops
    a = torch.from_numpy(synth.iid_images(8, 64, 64, c, 23)).cuda()
    b = torch.from_numpy(synth.iid_images(64, 64, 64, c, 24)).cuda()
    whole = ops.myrtle_nngp(a, b, depth, 2.0, sb2)
    assert bool(torch.isfinite(whole).all())
    for n1, n2 in ((1, 1), (1, 8), (2, 9), (1, 33), (2, 50), (4, 33), (3, 64)):
        print(f"64x64 depth {depth} {n1} x {n2}", flush=True)
        assert torch.equal(ops.myrtle_nngp(a[:n1].contiguous(), b[:n2].contiguous(), depth, 2.0, sb2), whole[:n1, :n2])
