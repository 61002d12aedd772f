"""FC NNGP blocks whose operands change places: K(x2, x1) is the transpose of
K(x1, x2) bit for bit in every kernel, so a Gram assembled block by block is
exactly symmetric (the conjugate-gradient solver takes it to be)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_05420_amd import ops
    return ops


def _rows(n, d, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    # (features of very different magnitude: every part of the products matters somewhere)
    return torch.randn((n, d), generator=gen, device="cuda") * torch.exp2(
        torch.randint(-12, 13, (1, d), generator=gen, device="cuda").float())


@pytest.mark.parametrize("n1,n2,d", [
    (5, 40, 70), (100, 333, 3072),                      # 16 x 16 tiles
    (900, 1000, 1), (900, 1000, 50), (900, 1000, 63),   # 64 x 64, all nine products
    (900, 1000, 64), (900, 1001, 333),                  # 64 x 64
    (3300, 3500, 384), (3333, 3301, 785),               # 128 x 128
])
@pytest.mark.parametrize("depth", [0, 3])
def test_exchanged_operands(nk, n1, n2, d, depth):
    print(f"fc {n1} x {n2} x {d} depth {depth}", flush=True)
    x1, x2 = _rows(n1, d, 71), _rows(n2, d, 72)
    assert torch.equal(nk.fc_nngp(x1, x2, depth, 2.0, 0.01), nk.fc_nngp(x2, x1, depth, 2.0, 0.01).t())


def test_gram_from_blocks(nk):
    print("fc gram of 3 x 3 blocks", flush=True)
    x = _rows(2100, 200, 73)
    cut = (0, 700, 1500, 2100)
    part = [x[a:b] for a, b in zip(cut, cut[1:])]
    k = torch.cat([torch.cat([nk.fc_nngp(a, None if a is b else b, 3, 2.0, 0.01) for b in part], 1) for a in part])
    assert torch.equal(k, k.t())
    whole = nk.fc_nngp(x, None, 3, 2.0, 0.01)
    d = whole.diagonal().sqrt()
    assert ((k - whole).abs() / (d[:, None] * d)).max() <= 1e-6  # (two float32 sums of 200 terms and three maps)
