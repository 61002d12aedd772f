"""The float64 products of the low-rank solvers are rounded once, however large
the neighbours of a term are.

K_rn K_nr is made diagonal: column j of K_nr is not zero in 64 rows of its own,
every 16th of them 1 (4 in all) and the others 2^-28, so each diagonal sum is 4 + 60
2^-56, whose float64 value is 4 + 2^-50.  With K_rr = -4 I, lambda = 1 and no jitter
the system's matrix is 2^-50 I, or 0, which is not positive definite, if the
small squares are lost beside the ones (a plain float64 sum loses them: the
first test)."""
import numpy as np
import pytest
import torch

ROWS = 64


def _column():
    k = np.full(ROWS, 2.0 ** -28, dtype=np.float32)
    k[::16] = 1.0
    return k


def test_a_plain_sum_loses_them():
    s = 0.0
    for v in _column().astype(np.float64):
        s += v * v
    assert s == 4.0
    import fractions

    exact = sum(fractions.Fraction(float(v)) ** 2 for v in _column())
    assert float(exact) == 4.0 + 2.0 ** -50


def _problem(r, c, scale):
    """r such columns, column j scaled by scale[j] (a power of two), and targets
    with K_rn Y = 1 in column j of row j mod c."""
    k_nr = torch.zeros((r * ROWS, r), device="cuda")
    col = torch.from_numpy(_column()).cuda()
    for j in range(r):
        k_nr[j * ROWS:(j + 1) * ROWS, j] = col * scale[j]
    k_rr = torch.diag(-4.0 * torch.as_tensor(scale, device="cuda", dtype=torch.float32) ** 2)
    y = torch.zeros((r * ROWS, c), device="cuda")
    for j in range(r):
        y[j * ROWS, j % c] = 1.0 / scale[j]
    return k_nr, k_rr, y


@pytest.mark.gpu
@pytest.mark.parametrize("r,c", [(1, 1), (3, 2), (17, 1), (40, 3), (200, 10), (720, 2)])
@pytest.mark.parametrize("scaled", [False, True])
def test_normal_matrix(r, c, scaled):
    from paper_2303_05420_amd import ops

    print(f"SoR with {r} columns, scaled {scaled}", flush=True)
    scale = [2.0 ** ((7 * j) % 40 - 20) if scaled else 1.0 for j in range(r)]
    k_nr, k_rr, y = _problem(r, c, scale)
    # v = (2^-50 scale^2)^{-1}, read out by K_mr = 2^-50 scale^2
    k_mr = torch.diag(torch.as_tensor([2.0 ** -50 * s * s for s in scale], device="cuda", dtype=torch.float32))
    pred = ops.krr_sor(k_nr, k_rr, k_mr, y, 1.0, 0.0)
    want = torch.zeros((r, c), device="cuda")
    for j in range(r):
        want[j, j % c] = 1.0
    assert torch.equal(pred, want)
