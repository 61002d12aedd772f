"""The float64 factorisation, substitutions and products of the ridge
solvers at the edges of their tiles (16, 32 and 64), through the entry points
that use them, against the float64 oracle.

Tolerances: predictions come out in float32 (6e-8 of the largest, rounding)
after float64 solves whose error is about cond(A) * 2.2e-16; the systems here
have condition numbers below 1e9 (the normal equations of the low-rank
methods: the square of a largest eigenvalue of about 700, over lambda *
jitter = 1e-3), so 1e-6 of the largest prediction holds both."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import approx

pytestmark = pytest.mark.gpu

TOL = 1e-6


@pytest.fixture(scope="module")
def nk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_05420_amd import ops
    return ops


def _gpu(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


def _problem(n, m, c, seed=51):
    x = synth.correlated_images(n + m, 8, 8, 3, 3.0, seed).reshape(n + m, -1)
    k = oracle.fc_nngp(x, x).astype(np.float32)
    y = np.random.default_rng(seed).standard_normal((n, c)).astype(np.float32)
    return k[:n, :n].copy(), k[n:, :n].copy(), k[n:, n:].copy(), y


def _close(got, want):
    err = np.max(np.abs(got.cpu().numpy() - want)) / np.max(np.abs(want))
    print(f"  relative error {err:.2e}", flush=True)
    assert err <= TOL


@pytest.mark.parametrize("n,m,c", [(1, 1, 1), (15, 3, 2), (16, 17, 16), (63, 1, 17), (64, 33, 1), (65, 16, 3),
                                   (128, 2, 70), (129, 5, 10), (193, 64, 16), (400, 300, 33)])
def test_direct_solve(nk, n, m, c):
    k, kt, _, y = _problem(n, m, c)
    print(f"krr {n} x {m} x {c}", flush=True)
    _close(nk.krr_predict(_gpu(k), _gpu(kt), _gpu(y), 1e-3), oracle.krr_predict(k, kt, y, 1e-3))


def test_direct_solve_not_positive_definite(nk):
    """A pivot that is not positive in the last panel is reported."""
    n = 130
    k = np.eye(n, dtype=np.float32)
    k[n - 1, n - 1] = -1.0
    with pytest.raises(RuntimeError):
        nk.krr_predict(_gpu(k), _gpu(k[:2]), _gpu(np.ones((n, 1))), 0.0)


@pytest.mark.parametrize("n,r,m,c", [(20, 1, 1, 1), (65, 33, 15, 2), (300, 64, 17, 16), (700, 257, 3, 17),
                                     (600, 530, 33, 5)])
def test_low_rank(nk, n, r, m, c):
    k, kt, _, y = _problem(n, m, c)
    lam, jit = 1e-1, 1e-2
    print(f"low rank {n} x {r} x {m} x {c}", flush=True)
    args = (_gpu(k[:, :r]), _gpu(k[:r, :r]))
    _close(nk.krr_nystrom(*args, _gpu(kt), _gpu(y), lam, jit),
           approx.nystrom_predict(k[:, :r], k[:r, :r], kt, y, lam, jit))
    _close(nk.krr_sor(*args, _gpu(kt[:, :r]), _gpu(y), lam, jit),
           approx.sor_predict(k[:, :r], k[:r, :r], kt[:, :r], y, lam, jit))


@pytest.mark.parametrize("sizes,m,c", [((1, 2), 1, 1), ((64, 65, 63), 16, 3), ((150, 70), 65, 17)])
def test_blocks(nk, sizes, m, c):
    n = sum(sizes)
    k, kt, ktt, y = _problem(n, m, c)
    cut = np.cumsum((0,) + sizes)
    rng = [slice(a, b) for a, b in zip(cut[:-1], cut[1:])]
    blocks = [k[s, s] for s in rng]
    print(f"blocks {sizes} x {m} x {c}", flush=True)
    gb = [_gpu(b) for b in blocks]
    kmi, yi = [kt[:, s] for s in rng], [y[s] for s in rng]
    _close(nk.krr_block_diag(gb, _gpu(kt), _gpu(y), 1e-1), approx.block_diag_predict(blocks, kmi, yi, 1e-1))
    _close(nk.krr_bcm(gb, _gpu(kt), _gpu(ktt), _gpu(y), 1e-1, 1e-1),
           approx.bcm_predict(blocks, kmi, yi, ktt, 1e-1, 1e-1))
