"""Products with the Gram matrix on either side of the rule that splits its rows
by the number of columns and rows, against float64.

Tolerance: a float64 sum of n products in any order is off by at most n 2^-53 of
the sum of their magnitudes."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 300, 8191, 8193, 9001])
@pytest.mark.parametrize("c", [1, 7, 8, 10, 13, 14, 16])
def test_products(n, c):
    from paper_2303_05420_amd import ops

    print(f"K.P {n} rows, {c} columns", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(101)
    k = torch.randn((n, n), generator=gen, device="cuda")
    k = torch.triu(k) + torch.triu(k, 1).t()
    p = torch.randn((n, c), generator=gen, dtype=torch.float64, device="cuda")
    q = ops.gram_matvec(k, p, 0.25)
    d = k.double()
    assert ((q - (d @ p + 0.25 * p)).abs() <= 2 * n * 2.0 ** -53 * (d.abs() @ p.abs() + p.abs())).all()
    assert torch.equal(q, ops.gram_matvec(k, p, 0.25))
