"""FC NNGP blocks at the edges of its kernels: few outputs (16 x 16 tiles),
64 x 64 and 128 x 128 tiles of split products, feature counts around a tile's
depth, rows that start at any element, padded output rows, and non-finite
inputs.

Tolerance 1e-6 normalised (|K - K_ref| / sqrt(K(x,x) K(x',x'))): float32 dot
products of d normalised terms (below 2^-24 sqrt(d / 16) each, 8e-7 at the
largest d here), the float32 diagonals and three ReLU maps (1.3e-7 each, which
the recursion does not amplify)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-6


@pytest.fixture(scope="module")
def nk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_05420_amd import ops
    return ops


def _rows(n, d, seed, offset=0):
    """n x d normal rows whose memory starts `offset` floats past an allocation."""
    x = np.random.default_rng(seed).standard_normal((n, d)).astype(np.float32)
    flat = torch.empty(n * d + offset, device="cuda")
    view = flat[offset:].view(n, d)
    view.copy_(torch.from_numpy(x))
    return x, view


def _check(k, x1, x2, pick1, pick2, depth):
    ref = oracle.fc_nngp(x1[pick1], x2[pick2], depth, 2.0, 0.01)
    d1 = np.array([oracle.fc_nngp(x1[i:i + 1], x1[i:i + 1], depth, 2.0, 0.01)[0, 0] for i in pick1])
    d2 = np.array([oracle.fc_nngp(x2[i:i + 1], x2[i:i + 1], depth, 2.0, 0.01)[0, 0] for i in pick2])
    got = k[torch.as_tensor(pick1, device="cuda")][:, torch.as_tensor(pick2, device="cuda")].cpu().numpy()
    err = np.max(np.abs(got - ref) / np.sqrt(np.outer(d1, d2)))
    print(f"  normalised error {err:.2e}", flush=True)
    assert err <= TOL


def _edges(n):
    return sorted({0, 1, 15, 16, 31, 32, 63, 64, 65, 127, 128, n // 2, n - 17, n - 2, n - 1} & set(range(n)))


@pytest.mark.parametrize("n1,n2,d,offset", [
    (1, 1, 1, 0), (17, 3, 15, 1), (16, 33, 16, 2), (5, 100, 17, 3), (30, 250, 255, 1), (3, 40, 256, 0), (18, 5, 3071, 1),
    (700, 610, 1, 1), (641, 640, 15, 0), (640, 700, 16, 3), (650, 640, 17, 1), (640, 640, 63, 2), (640, 641, 64, 1),
    (655, 640, 65, 3), (640, 640, 192, 0), (3300, 3333, 384, 1), (3300, 3200, 400, 0), (3201, 3300, 385, 2),
])
def test_blocks(nk, n1, n2, d, offset):
    print(f"fc {n1} x {n2} x {d}, rows at {offset}", flush=True)
    x1, g1 = _rows(n1, d, 61, offset)
    x2, g2 = _rows(n2, d, 62, offset)
    big = torch.full((n1, n2 + 3), float("nan"), device="cuda")
    k = nk.fc_nngp(g1, g2, 3, 2.0, 0.01, out=big[:, :n2])
    assert torch.isfinite(k).all() and torch.isnan(big[:, n2:]).all()
    _check(k, x1, x2, _edges(n1), _edges(n2), 3)


@pytest.mark.parametrize("n,d,pad", [(1, 4, 0), (300, 33, 1), (900, 63, 0), (901, 130, 3), (902, 64, 2), (4610, 384, 0)])
def test_symmetric_blocks(nk, n, d, pad):
    print(f"fc symmetric {n} x {d}, ldk {n + pad}", flush=True)
    x, g = _rows(n, d, 63)
    big = torch.full((n, n + pad), float("nan"), device="cuda")
    k = nk.fc_nngp(g, None, 3, 2.0, 0.01, out=big[:, :n])
    assert torch.isfinite(k).all() and torch.equal(k, k.t())
    assert pad == 0 or torch.isnan(big[:, n:]).all()
    _check(k, x, x, _edges(n), _edges(n), 3)


@pytest.mark.parametrize("n,d", [(20, 70), (700, 70), (700, 20), (3300, 400)])
@pytest.mark.parametrize("depth", [0, 2])
def test_non_finite_rows(nk, n, d, depth):
    """An infinity (or NaN, or a row whose square overflows) touches only its
    own row and column, which hold what float32 arithmetic of the recursion
    gives: without a ReLU layer the plain dot product."""
    x, g = _rows(n, d, 64)
    y, h = _rows(n, d, 65)
    clean = nk.fc_nngp(g, h, depth, 2.0, 0.01).clone()
    g[3, 1], g[5, 0], g[7, 2] = float("inf"), float("nan"), 3e38
    h[:, 1] = h[:, 1].abs() + 0.5  # (the infinity's products are +inf)
    want = nk.fc_nngp(g[8:].contiguous(), h, depth, 2.0, 0.01)
    k = nk.fc_nngp(g, h, depth, 2.0, 0.01)
    print(f"fc non-finite {n} x {d} depth {depth}", flush=True)
    assert torch.allclose(k[8:], want, rtol=1e-5, atol=1e-6) and torch.isfinite(k[:3]).all()
    assert torch.isfinite(clean).all()
    if depth == 0:
        dot = (g[7].double() @ h.double().t()).float() * 2.0 / d + 0.01  # (float32: it overflows where the kernel does)
        assert torch.isposinf(k[3]).all() and torch.isnan(k[5]).all()
        assert torch.allclose(k[7], dot, rtol=1e-5)
    else:
        assert torch.isnan(k[3]).all() and torch.isnan(k[7]).all()
