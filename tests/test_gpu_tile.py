"""Value scan of the wave path (nx >= 5) on elements whose I + C J systems need row exchanges.

The scan inverts I + J C without row exchanges and repeats with partial pivoting when a multiplier
is large; solved problems do not get there, so the elements here are drawn: C and J are rank-one
heavy positive semidefinite matrices with large off-diagonal entries.  Reference: the sequential
fold in 64 bits with numpy's solver."""
import numpy as np
import pytest
import torch

from helpers import relerr
from lqt_layout import dense_to_soa
from paper_2212_11744_amd import lqt

pytestmark = pytest.mark.gpu


def _elements(rng, nx, T):
    def psd():
        x = rng.standard_normal((T, nx, 1))
        y = rng.standard_normal((T, nx, 2))
        return 0.8 * x @ x.transpose(0, 2, 1) + 0.02 * y @ y.transpose(0, 2, 1)

    A = 0.5 * rng.standard_normal((T, nx, nx)) / np.sqrt(nx)
    return {"A": A, "b": rng.standard_normal((T, nx)), "C": psd(),
            "eta": rng.standard_normal((T, nx)), "J": psd()}


def _largest_multiplier(M):
    """Of elimination without row exchanges."""
    M, worst = M.copy(), 0.0
    for c in range(M.shape[0] - 1):
        f = M[c + 1:, c] / M[c, c]
        worst = max(worst, np.max(np.abs(f)))
        M[c + 1:] -= f[:, None] * M[c]
    return worst


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-9), (torch.float32, 1e-4)])
@pytest.mark.parametrize("nx", [5, 8, 9, 16])
@pytest.mark.parametrize("T", [4, 7, 38])
def test_scan_needing_row_exchanges(nx, T, dtype, tol):
    rng = np.random.default_rng(100 * nx + T)
    el = _elements(rng, nx, T)
    if dtype == torch.float32:  # the reference folds what the scan reads
        el = {k: a.astype(np.float32).astype(np.float64) for k, a in el.items()}
    Qf, rf = el["J"][0].copy(), el["b"][0].copy()
    S, v, worst = [Qf], [Qf @ rf], 0.0
    for k in range(T - 1, -1, -1):
        A, b, C, e, J = (el[q][k] for q in ("A", "b", "C", "eta", "J"))
        M = np.eye(nx) + C @ S[-1]
        worst = max(worst, _largest_multiplier(M.T))
        P = np.linalg.solve(M, A)
        w = v[-1] - S[-1] @ b
        S.append(P.T @ S[-1] @ A + J)
        S[-1] = 0.5 * (S[-1] + S[-1].T)
        v.append(P.T @ w + e)
    assert T < 38 or worst > 4.0  # the elements do reach the pivoted inverse
    to = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")
    z = np.zeros
    p = lqt.DeviceProblem(nx, 1, T, 1, 1, dtype, to(z((1, T + 1))), to(z((nx, nx))), to(z((nx, 1))),
                          to(z((1, nx, nx))), to(np.ones((1, 1, 1))), to(z((1, 2 * T + 1, nx))),
                          to(Qf[None]), to(rf[None]), to(z((1, nx))))
    got = lqt.scan_value(p, to(dense_to_soa(el, nx, Ad=el["A"] - np.eye(nx))[None]))
    torch.cuda.synchronize()
    assert relerr(got[0][0].cpu(), np.stack(S[::-1])) < tol
    assert relerr(got[1][0].cpu(), np.stack(v[::-1])) < tol
