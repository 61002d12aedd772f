"""Ridge solves of systems far from well conditioned (points that nearly
coincide in groups of the size of the blocks the factorisation inverts),
against float64 with iterative refinement in extended precision.

Tolerance: float32 predictions, 6e-8 of the largest, after a backward stable
float64 solve: condition times 4 n 2^-53."""
import numpy as np
import pytest
import scipy.linalg as sl
import torch

pytestmark = pytest.mark.gpu


def _kernel(a, b):
    return np.exp(-((a[:, None] - b[None]) ** 2).sum(-1) / a.shape[1]).astype(np.float32)


@pytest.mark.parametrize("n,group,spread,ridge", [(200, 16, 1e-2, 1e-6), (450, 15, 1e-3, 1e-6), (450, 64, 1e-3, 1e-5),
                                                  (300, 3, 1e-4, 1e-6)])
def test_near_duplicates(n, group, spread, ridge):
    from paper_2303_05420_amd import ops

    rng = np.random.default_rng(121)
    base = rng.standard_normal((n // group + 1, 20))
    x = np.repeat(base, group, 0)[:n] + spread * rng.standard_normal((n, 20))
    t = base[rng.integers(0, base.shape[0], 40)] + 0.3 * rng.standard_normal((40, 20))
    k, kt = _kernel(x, x), _kernel(t, x)
    k = np.maximum(k, k.T)
    y = rng.standard_normal((n, 4)).astype(np.float32)
    a = k.astype(np.float64) + ridge * np.mean(np.diag(k).astype(np.float64)) * np.eye(n)
    eig = np.linalg.eigvalsh(a)
    cond = eig[-1] / eig[0]
    assert eig[0] > 0 and cond > 1e5
    f = sl.cho_factor(a, lower=True)
    wide = a.astype(np.longdouble)
    sol = sl.cho_solve(f, y.astype(np.float64)).astype(np.longdouble)
    for _ in range(20):
        sol += sl.cho_solve(f, (y.astype(np.longdouble) - wide @ sol).astype(np.float64))
    want = (kt.astype(np.longdouble) @ sol).astype(np.float64)
    gpu = lambda v: torch.from_numpy(v).cuda()
    got = ops.krr_predict(gpu(k), gpu(kt), gpu(y), ridge).cpu().numpy()
    err = np.max(np.abs(got - want)) / np.max(np.abs(want))
    print(f"condition {cond:.1e}: error {err:.2e}", flush=True)
    # (the cancellation of kt sol is part of it: |kt| |sol| against the prediction)
    grow = np.max(np.abs(kt).astype(np.float64) @ np.abs(sol).astype(np.float64)) / np.max(np.abs(want))
    assert err <= 6e-8 + 4 * n * 2.0 ** -53 * cond * grow
