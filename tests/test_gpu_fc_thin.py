"""FC NNGP blocks of a few rows against many columns stay in the kernel for few
outputs however long they get: an entry has the bits it has in a short block."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_05420_amd import ops
    return ops


@pytest.mark.parametrize("n1,n2,d", [(1, 24577, 70), (4, 60001, 33), (16, 25600, 100), (16, 100000, 17)])
def test_thin_blocks(nk, n1, n2, d):
    print(f"fc {n1} x {n2} x {d}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(91)
    x1, x2 = (torch.randn((n, d), generator=gen, device="cuda") for n in (n1, n2))
    k = nk.fc_nngp(x1, x2, 3, 2.0, 0.01)
    pick = [0, 15, 16, n2 // 2, n2 - 17, n2 - 1]
    few = nk.fc_nngp(x1, x2[pick].contiguous(), 3, 2.0, 0.01)
    assert torch.equal(k[:, pick], few)
    assert torch.equal(nk.fc_nngp(x2, x1, 3, 2.0, 0.01), k.t())
    a, b = x1.cpu().numpy(), x2[pick].cpu().numpy()
    ref = oracle.fc_nngp(a, b, 3, 2.0, 0.01)
    d1 = np.array([oracle.fc_nngp(r[None], r[None], 3, 2.0, 0.01)[0, 0] for r in a])
    d2 = np.array([oracle.fc_nngp(r[None], r[None], 3, 2.0, 0.01)[0, 0] for r in b])
    # (float32 sums of at most 100 terms, the diagonals and three maps of 1.3e-7)
    assert np.max(np.abs(few.cpu().numpy() - ref) / np.sqrt(np.outer(d1, d2))) <= 1e-6
