"""Solves under a terminal weight Qf = w I that is large against the running cost, on the tree kernels.

The systems I + C S then reach a size of w, so that a solve in working precision eps leaves the
trajectory a relative error of eps w times a small factor: the tolerance is 100 eps w.  A combination
that forms M^{-1} C as C minus nearly all of it is off by eps w^2.  S and v, which are computed from
the value at the right end without such a factor in their largest entries, stay within 100 eps.
Reference: the sequential fold of the elements the call returns, in extended precision."""
import numpy as np
import pytest
import torch

from lqt_layout import soa_to_dense
from paper_2212_11744_amd import lqt
from paper_2212_11744_amd import workloads as W

pytestmark = pytest.mark.gpu

LD = np.longdouble


def _solve(M, B):
    M, B = M.copy(), B.copy()
    for c in range(M.shape[0]):
        q = c + np.argmax(np.abs(M[c:, c]))
        M[[c, q]], B[[c, q]] = M[[q, c]], B[[q, c]]
        B[c], M[c] = B[c] / M[c, c], M[c] / M[c, c]
        for i in range(M.shape[0]):
            if i != c:
                B[i], M[i] = B[i] - M[i, c] * B[c], M[i] - M[i, c] * M[c]
    return B


def _reference(el, Qf, rf, x0):
    T, nx = el["b"].shape
    A, b, C, e, J = (el[k].astype(LD) for k in ("Ad", "b", "C", "eta", "J"))
    I = np.eye(nx, dtype=LD)
    S, v, maps = [Qf], [Qf @ rf], []
    for k in range(T - 1, -1, -1):
        X = _solve(I + C[k] @ S[-1], np.concatenate([I + A[k], (b[k] + C[k] @ v[-1])[:, None]], 1))
        P = X[:, :nx]
        w = v[-1] - S[-1] @ b[k]
        S.append(J[k] + P.T @ (S[-1] @ (I + A[k])))
        v.append(e[k] + P.T @ w)
        maps.append((P, X[:, nx]))
    x = [x0]
    for P, q in reversed(maps):
        x.append(P @ x[-1] + q)
    return {"S": np.array(S[::-1]), "v": np.array(v[::-1]), "x": np.array(x)}


@pytest.mark.parametrize("nx", [4, 6, 8, 10, 16])
@pytest.mark.parametrize("dtype,weight", [(torch.float64, 1e3), (torch.float64, 1e6),
                                          (torch.float32, 1e2)])
def test_heavy_terminal_weight(nx, dtype, weight):
    T = 64
    p = W.point_mass(nx, T, 4, d=nx // 2)
    p.Qf = weight * np.eye(nx)
    dp = lqt.DeviceProblem.from_problems([p], dtype=dtype)
    got = lqt.solve(dp, keep_elements=True)
    torch.cuda.synchronize()
    ld = lambda a: a[0].double().cpu().numpy().astype(LD)
    ref = _reference(soa_to_dense(got["elts"][0].double().cpu().numpy(), nx, T), ld(dp.Qf),
                     ld(dp.rf), ld(dp.x0))
    eps = torch.finfo(dtype).eps
    for k, tol in (("S", 100 * eps), ("v", 100 * eps), ("x", 100 * eps * weight)):
        e = float(np.max(np.abs(ld(got[k]) - ref[k])) / np.max(np.abs(ref[k])))
        assert e < tol, f"{k}: {e:.3e} against {tol:.3e}"
