"""FC NNGP blocks on rows whose features take few distinct values: the parts of
a product that the split leaves out then have one sign throughout the sum.

Tolerance (normalised, no ReLU layer): what a sum by fp32 matrix instructions may
be off, a rounding of 2^-24 of the sum per four terms, and four more for the
parts left out, the diagonal, the scale and the result."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_05420_amd import ops
    return ops


@pytest.mark.parametrize("values", [1, 2, 3])
@pytest.mark.parametrize("n,d", [(60, 200), (700, 40), (700, 64), (700, 1000), (3300, 400), (3300, 3072)])
def test_few_valued_rows(nk, n, d, values):
    print(f"fc {n} x {d}, rows of {values} values", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(81 + values)

    def rows():
        v = torch.randn((n, values), generator=gen, device="cuda")
        return torch.gather(v, 1, torch.randint(0, values, (n, d), generator=gen, device="cuda"))

    x1, x2 = rows(), rows()
    k = nk.fc_nngp(x1, x2, 0, 2.0, 0.0)
    a, b = x1.double(), x2.double()
    want = 2.0 * (a @ b.t().contiguous()) / d
    scale = torch.sqrt((2.0 * a.square().sum(1) / d)[:, None] * (2.0 * b.square().sum(1) / d))
    err = float(((k.double() - want).abs() / scale).max())
    bound = (d / 4 + 4) * 2.0 ** -24
    print(f"  error {err:.2e}, bound {bound:.2e}", flush=True)
    assert err <= bound
