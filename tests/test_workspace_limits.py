"""Workspaces that callers sized for an earlier form of the conjugate-gradient
solver's plan are still large enough: its size never grows past what these
formulas give (256-byte aligned regions in order)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2303_05420_amd import _lib


def _total(regions):
    at = 0
    for b in regions:
        at = (at + 255) // 256 * 256 + b
    return at + 256


def _splits(n):
    blocks = (n + 1023) // 1024
    return max(1, min((512 + blocks - 1) // blocks, (n + 63) // 64, 64))


def _pivots(n, rank):
    nb = (n + 255) // 256
    return [8 * n, 16 * nb, 8 * nb, 8 * max(rank, 1)]


def _solver(n, rank):
    r, g = max(rank, 1), 16
    groups = (rank + 63) // 64
    lt = 1 if rank <= 0 else max(1, min((512 + groups - 1) // groups, (n + 255) // 256))
    return (_pivots(n, rank) + [16, 4 * r, 8 * n * rank, 8 * n * rank, 8 * rank * rank, 16, 8 * r * g, 8 * lt * r * g]
            + [8 * n * g] * 5 + [8 * ((n + 63) // 64) * g, 56 * g, 8 * _splits(n) * n * g, 8 * ((n + 63) // 64) * g])


@pytest.mark.parametrize("rank", [0, 1, 50, 300])
def test_solver_workspace_does_not_grow(rank):
    lib = _lib.lib()
    cfg = _lib.PcgCfg()
    cfg.rank, cfg.max_iter, cfg.tol, cfg.pivot_tol = rank, 10, 1e-8, 0.0
    for n in [*range(1, 4400, 7), 5000, 8192, 12287, 12288, 16384, 24576, 32768, 65536, 100000]:
        need = lib.nk_workspace_size(_lib.NK_OP_PCG, ctypes.byref(cfg), n, 4)
        assert 0 < need <= _total(_solver(n, min(rank, n))), n


@pytest.mark.gpu
@pytest.mark.parametrize("n,rank", [(200, 20), (1030, 70), (2049, 33)])
def test_pivoted_cholesky_in_the_smaller_workspace(n, rank):
    """Pivot steps of 256 rows a workgroup choose what those of 64 rows choose."""
    from paper_2303_05420_amd import ops

    print(f"pivoted Cholesky {n}, rank {rank}", flush=True)
    x = np.random.default_rng(7).standard_normal((n, 40))
    k = torch.from_numpy(np.exp(-((x[:, None] - x[None]) ** 2).sum(-1) / 60).astype(np.float32)).cuda()
    full, piv, used = ops.pivoted_cholesky(k, rank)
    size = _total(_pivots(n, rank))
    assert size <= ops.workspace_size(_lib.NK_OP_PIVOTED_CHOL, None, n, rank)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    low = torch.zeros((rank, n), dtype=torch.float64, device="cuda")
    piv2 = torch.full((rank,), -1, dtype=torch.int32, device="cuda")
    got = ctypes.c_int32(0)
    stream = torch.cuda.current_stream().cuda_stream
    call = _lib.lib().nk_pivoted_cholesky
    _lib.check(call(k.data_ptr(), n, n, rank, 0.0, low.data_ptr(), piv2.data_ptr(), ctypes.byref(got), ws.data_ptr(),
                    size, stream))
    assert got.value == used == rank and torch.equal(piv, piv2)
    # (the sums over earlier columns in four parts or one: float64 rounding)
    assert (low.t() - full).abs().max() <= 1e-12
    assert call(k.data_ptr(), n, n, rank, 0.0, low.data_ptr(), piv2.data_ptr(), None, ws.data_ptr(), size - 256,
                stream) == _lib.NK_EINVAL


@pytest.mark.gpu
def test_solver_in_the_former_workspace():
    from paper_2303_05420_amd import ops

    n, rank, c = 2049, 40, 3
    print(f"conjugate gradients {n}, rank {rank}", flush=True)
    rng = np.random.default_rng(8)
    x = rng.standard_normal((n, 30))
    k = torch.from_numpy(np.exp(-((x[:, None] - x[None]) ** 2).sum(-1) / 60).astype(np.float32)).cuda()
    y = torch.from_numpy(rng.standard_normal((n, c))).cuda()
    cfg = _lib.PcgCfg()
    cfg.rank, cfg.max_iter, cfg.tol, cfg.pivot_tol = rank, 500, 1e-8, 0.0
    size = _total(_solver(n, rank))
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    out = torch.empty_like(y)
    _lib.check(_lib.lib().nk_krr_pcg(k.data_ptr(), n, n, y.data_ptr(), c, 1e-3, 1, ctypes.byref(cfg), out.data_ptr(), None,
                                     None, None, ws.data_ptr(), size, torch.cuda.current_stream().cuda_stream))
    want = ops.krr_pcg(k, y, 1e-3, rank=rank, tol=1e-8, max_iter=500)[0]
    assert torch.equal(out, want)
    lam = 1e-3 * float(k.diagonal().double().mean())
    res = y - (k.double() @ out + lam * out)
    assert (res.norm(dim=0) / y.norm(dim=0)).max() <= 1e-7
