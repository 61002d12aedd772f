"""GPU tests of the 32 x 32 CNN-VEC kernel, which takes the tables of a layer in
pieces of 8 rows through a ring of four in LDS, against the FP64 oracle:
depths at which the ring is not filled twice (1, 2) and at which it wraps (3, 9),
every channel count, with and without bias, pair blocks cut on either side,
and a symmetric block.  Bound: 2e-5 normalised, the one of every CNN-VEC block
(the fit of the map is good to 5e-6; the sums are of 3 x 3 terms)."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu
TOL = 2e-5


@pytest.mark.parametrize("n1,n2,C,depth,sb2,sym", [
    (1, 1, 3, 1, 0.01, False),
    (5, 3, 1, 1, 0.0, False),
    (3, 9, 2, 2, 0.01, False),
    (6, 6, 4, 3, 0.0, True),
    (7, 4, 3, 9, 0.0, False),
    (9, 9, 1, 9, 0.1, True),
])
def test_cv32_matches_oracle(n1, n2, C, depth, sb2, sym):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_05420_amd import ops
    print(f"cv 32x32x{C} depth {depth} {n1}x{n2} bias {sb2}", flush=True)
    xa = synth.iid_images(n1, 32, 32, C, 40 + n1)
    xb = xa if sym else synth.iid_images(n2, 32, 32, C, 60 + n2)
    ta = torch.from_numpy(xa).cuda()
    tb = None if sym else torch.from_numpy(xb).cuda()
    got = ops.cv_nngp(ta, tb, depth=depth, sigma_w2=2.0, sigma_b2=sb2).cpu().numpy()
    _, d1 = oracle.cv_self(xa, depth, 2.0, sb2)
    _, d2 = oracle.cv_self(xb, depth, 2.0, sb2)
    ref = oracle.cv_gram(xa, xb, depth, 2.0, sb2)
    assert np.max(np.abs(got - ref) / np.sqrt(np.outer(d1, d2))) <= TOL
    if sym:
        assert np.array_equal(got, got.T)
