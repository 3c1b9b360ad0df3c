"""sym_eigen at the edges of what its kernels tile: 64 column pairs by 8 row
pairs per workgroup, and the eigenvector kernel's variants, whose last sizes
are 512, 1,024, 2,048, 4,096 and 8,192 (rows of V in LDS, then in memory).

Every entry of V passes through one rotation per round, n - 1 rounds a sweep,
at most 4 roundings each, and 16 sweeps are more than these matrices take: the
residual and V's departure from orthogonality stay within
16 (n - 1) 4 2^-53 of the largest eigenvalue and of one."""
import ctypes

import pytest

import paper_2509_12086_amd as saq
from gpu_util import cuda, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _matrix(n, kind):
    g = torch.Generator(device=cuda()).manual_seed(n)
    if kind == "dense":
        B = torch.randn(n, n, dtype=torch.float64, device=cuda(), generator=g)
        return (B + B.T) / 2
    A = torch.diag(torch.arange(1, n + 1, dtype=torch.float64, device=cuda()))
    if kind == "near diagonal":
        B = torch.randn(n, n, dtype=torch.float64, device=cuda(), generator=g)
        A += 1e-6 * (B + B.T)
    else:   # pairs (i, n - 1 - i): one sweep
        i = torch.arange(n // 2, device=cuda())
        A[i, n - 1 - i] = A[n - 1 - i, i] = 3.0
    return A


@pytest.mark.parametrize("n,kind", [
    (3, "dense"), (15, "dense"), (16, "dense"), (17, "dense"), (127, "dense"), (128, "dense"),
    (130, "dense"), (511, "dense"), (512, "dense"), (513, "dense"), (514, "dense"),
    (1024, "dense"), (1025, "dense"), (2048, "near diagonal"), (2049, "near diagonal"),
    (4096, "near diagonal"), (4098, "near diagonal"), (8194, "pairs")])
def test_sym_eigen_edges(n, kind):
    A = _matrix(n, kind)
    say(f"sym_eigen n={n} {kind}")
    w, V = saq.sym_eigen(A)
    torch.cuda.synchronize()
    tol = 16 * (n - 1) * 4 * 2.0 ** -53
    scale = float(w.abs().max())
    res = float((A @ V - V * w[None, :]).abs().max()) / scale
    orth = float((V.T.contiguous() @ V - torch.eye(n, dtype=torch.float64, device=cuda())).abs().max())
    say(f"  residual {res:.1e} orthogonality {orth:.1e} (within {tol:.1e})")
    assert res < tol and orth < tol


@pytest.mark.parametrize("n", [4, 5, 6, 8, 59, 60, 61, 62, 63, 64, 65, 123, 124, 125, 126, 187, 240, 250])
def test_sym_eigen_pair_tiles(n):
    """Around the 30 row and 62 column pairs that a workgroup takes through two
    rounds at once."""
    test_sym_eigen_edges(n, "dense")


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 16, 17, 21, 22, 23, 24, 25, 63, 64, 65, 130, 333, 514])
@pytest.mark.parametrize("shift", [0, 1])
def test_sym_eigen_workspace(n, shift):
    """Three n x n buffers (of an even n) and what little the convergence test
    takes are enough, nothing past them or V is touched, V may start at any
    double, and the result does not depend on it."""
    A = _matrix(n, "dense")
    w0, V0 = saq.sym_eigen(A)
    N = n + n % 2
    ws_bytes = 3 * ((N * N * 8 + 255) // 256 * 256) + 65536
    assert saq.lib().saq_sym_eigen_workspace_bytes(n) <= ws_bytes
    ws = torch.full((ws_bytes + 4096,), 0x5a, dtype=torch.uint8, device=cuda())
    buf = torch.full((n * n + 64,), 7.0, dtype=torch.float64, device=cuda())
    w = torch.empty(n, dtype=torch.float64, device=cuda())
    say(f"sym_eigen n={n} V {8 * shift} bytes off")
    V = buf[2 + shift:2 + shift + n * n]
    P = ctypes.c_void_p
    rc = saq.lib().saq_sym_eigen_device(P(A.data_ptr()), n, P(w.data_ptr()), P(V.data_ptr()), P(ws.data_ptr()),
                                        ws_bytes, P(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert rc == 0
    assert torch.equal(w, w0) and torch.equal(V.view(n, n), V0)
    assert bool((buf[:2 + shift] == 7.0).all()) and bool((buf[2 + shift + n * n:] == 7.0).all())
    assert bool((ws[ws_bytes:] == 0x5a).all())
