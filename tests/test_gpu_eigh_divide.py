"""The eigendecomposition on matrices that exercise the divide and conquer's deflation and its sizes (first-level pairs
and single indices, where the matrices lie, LDS pitches): eigenvalues, orthogonality and reconstruction to rounding."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2512_23353_amd import isopo

pytestmark = pytest.mark.gpu


def _matrix(kind, m, rng):
    if kind == "gram":
        J = rng.standard_normal((m, 2 * m))
        return J @ J.T
    if kind == "identity":
        return np.eye(m)
    if kind == "low_rank":
        J = rng.standard_normal((m, max(1, m // 3)))
        return J @ J.T
    if kind == "toeplitz":                                # tridiagonal, every coupling alike
        return 2 * np.eye(m) - np.eye(m, k=1) - np.eye(m, k=-1)
    if kind == "wilkinson":                               # pairs of eigenvalues that agree to many digits
        return np.diag(np.abs(np.arange(m) - (m - 1) / 2)) + np.eye(m, k=1) + np.eye(m, k=-1)
    if kind == "blocks":                                  # equal blocks, weakly coupled: many equal poles
        b = 2 * np.eye(m) + 0.5 * (np.eye(m, k=1) + np.eye(m, k=-1))
        cut = np.arange(4, m - 1, 5)
        b[cut, cut + 1] = b[cut + 1, cut] = 1e-7
        return b
    if kind == "graded":
        s = 10.0 ** -np.linspace(0, 12, m)
        J = rng.standard_normal((m, 2 * m)) * s[:, None]
        return J @ J.T
    if kind == "duplicates":                              # pairs of equal sequences
        J = rng.standard_normal((m, 2 * m))
        J[1::2] = J[0:m - m % 2:2]
        return J @ J.T
    raise ValueError(kind)


@pytest.mark.parametrize("kind", ["gram", "identity", "low_rank", "toeplitz", "wilkinson", "blocks", "graded", "duplicates"])
@pytest.mark.parametrize("m", [1, 2, 3, 5, 6, 7, 17, 31, 33, 49, 63, 65, 97, 113, 115, 127, 129, 255, 257])
def test_divide_and_conquer(gpu_device, kind, m):
    K = _matrix(kind, m, np.random.default_rng(m)).astype(np.float32)
    K = (K + K.T) / 2
    D, U, info = isopo.ntk_eigh(torch.from_numpy(np.stack([K, 3 * K])).to(gpu_device))
    assert info.tolist() == [0, 0]
    for b, f in enumerate((1.0, 3.0)):
        Kd = (np.float32(f) * K).astype(np.float64)
        Dh, Uh = D[b].cpu().numpy(), U[b].cpu().numpy()
        ref = np.linalg.eigvalsh(Kd)
        # backward stable: a modest multiple of n rounding errors of the norm
        tol = 16 * (m + 8) * 2.0 ** -53
        size = max(np.abs(ref).max(), 1e-300)
        assert (np.diff(Dh) >= 0).all()
        assert np.abs(Dh - ref).max() <= tol * size
        assert np.abs(Uh.T @ Uh - np.eye(m)).max() <= tol
        assert np.abs((Uh * Dh) @ Uh.T - Kd).max() <= tol * size


@pytest.mark.parametrize("m", [3, 40, 150])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_non_finite_entries_are_reported(gpu_device, m, value):
    K = torch.eye(m, device=gpu_device).repeat(2, 1, 1)
    K[0, m // 2, 0] = K[0, 0, m // 2] = value
    D, U, info = isopo.ntk_eigh(K)
    assert info.tolist() == [1, 0] and torch.isfinite(D[1]).all() and not torch.isfinite(D[0]).any()


@pytest.mark.parametrize("m", [24, 40, 64, 90, 100, 128, 200])
def test_copies_of_sequences(gpu_device, m):
    """Rank-one matrices of whole numbers, alone and below a block 10^80 times as large: the trailing block of the reduction
    is rounding, of rank one again, and shrinks by a factor of 10^16 every few columns until squares underflow."""
    rng = np.random.default_rng(4)
    K = np.zeros((64, m, m))
    for k in range(0, 64, 2):
        a = rng.integers(1, 1 + rng.choice([1, 2, 4, 9]), m) * rng.choice([-1, 1], m)
        K[k] = np.outer(a, a)
        K[k + 1, :4, :4] = np.eye(4) * 2.0 ** 126
        K[k + 1, 4:, 4:] = np.outer(a, a)[4:, 4:] * (rng.integers(1, 50) * 2.0 ** -149)
    K = K.astype(np.float32)
    D, U, info = isopo.ntk_eigh(torch.from_numpy(K).to(gpu_device))
    assert not info.any()
    D, U, Kd = D.cpu().numpy(), U.cpu().numpy(), K.astype(np.float64)
    ref = np.linalg.eigvalsh(Kd)
    tol, size = 16 * (m + 8) * 2.0 ** -53, np.abs(ref).max(axis=1)
    assert (np.abs(D - ref).max(axis=1) <= tol * size).all()
    for b in range(len(K)):
        assert np.abs(U[b].T @ U[b] - np.eye(m)).max() <= tol
        assert np.abs((U[b] * D[b]) @ U[b].T - Kd[b]).max() <= tol * size[b]


def _eigh_in_steps(K, steps):
    """isopo_ntk_eigh with its limit on the steps per root as an argument (the library's internal C++ function)."""
    b, m, _ = K.shape
    D = torch.empty((b, m), dtype=torch.float64, device=K.device)
    U = torch.empty((b, m, m), dtype=torch.float64, device=K.device)
    info = torch.full((b,), -1, dtype=torch.int32, device=K.device)
    ws = isopo.alloc_workspace(isopo.load().isopo_ntk_eigh_workspace(m, b), K.device)
    fn = isopo.load()._ZN5isopo15launch_ntk_eighEPKfiiPdS2_PiPvP12ihipStream_ti
    ptr, num = ctypes.c_void_p, ctypes.c_int
    assert fn(ptr(K.data_ptr()), num(m), num(b), ptr(D.data_ptr()), ptr(U.data_ptr()), ptr(info.data_ptr()),
              ptr(ws.data_ptr()), ptr(torch.cuda.current_stream().cuda_stream), num(steps)) == 0
    return D, U, info.tolist()


@pytest.mark.parametrize("m", [3, 20, 64, 100, 130, 300])
def test_roots_that_do_not_converge_are_reported(gpu_device, m):
    """One step per root is too few for a Gram matrix and enough for a diagonal one, which has none to find; a tenth of the
    library's own limit is enough for all."""
    rng = np.random.default_rng(m)
    K = np.stack([_matrix("gram", m, rng), np.diag(np.arange(1.0, m + 1)), _matrix("duplicates", m, rng)])
    K = torch.from_numpy(K.astype(np.float32)).to(gpu_device)
    assert _eigh_in_steps(K, 1)[2][:2] == [1, 0]
    D, U, info = _eigh_in_steps(K, 10)
    assert info == [0, 0, 0]
    D1, U1, info = isopo.ntk_eigh(K)
    assert info.tolist() == [0, 0, 0] and torch.equal(D, D1) and torch.equal(U, U1)
