"""The block steps on the GPU against the fp64 oracle at the sizes where their
launches change: pivot blocks of the 64x64 inverse (widths around multiples
of 16), the U-step's column groups (few rows, many columns), the V-step's row
groups (one from 8225 columns on, also in wide blocks), a contraction with fewer K steps than
waves or a remainder of them, and wide blocks of 2, 3 and 4 quarters with a
last quarter of 1 or 64 components.

Tolerances.  The contractions are exact for the residual rounded to fixed
point.  V-step: column j's unit is at most 2^-29 ||R_:j||, so an entry moves by
at most 2^-30 ||R_:j|| and
    |P - U^T R|_cj <= 2^-30 (sum_i |U_ic|) ||R_:j||,
which |G^-1| carries to Y.  U-step: row i's unit is at most
2^-29 max_j |R_ij h_j| (a measured bound may exceed the maximum by a factor
below 2: doubled), so
    |Q - R diag(h) V|_ic <= 2^-29 (sum_j |V_jc|) max_j |R_ij h_j|.
The fp64 inverse and the product with it: 8 bb cond(G) 2^-53 of the largest
entry of the result.  The weighted Gram takes each weight to within
2^-42 max h, so G moves by at most dG = 2^-42 max h |V|^T |V| (its ridge by
less) and Z = Q G^-1 by |Z| dG |G^-1| to first order, doubled.  Trits: bit-exact against T_tau of the GPU's own targets
outside the threshold band.  Deflation: one fp32 rounding per quarter and the
fp32 sums of its 3 x 64 terms, 2e-6 of sum_c |U_ic d_c V_jc| + |R_ij| each.
"""
import numpy as np
import pytest

import oracle
from paper_2607_13511_amd import synth
from test_gpu_parity import cols_parity, cuda, host

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# m, n, bb
NARROW = [(33, 2051, 5), (37, 40, 1), (97, 4100, 16), (97, 4100, 17), (250, 700, 48), (1030, 517, 63), (700, 1500, 64),
          (70, 8225, 24), (3100, 130, 33)]
WIDE = [(700, 130, 65), (419, 999, 128), (1100, 523, 129), (805, 1290, 193), (1025, 811, 256), (300, 8230, 130)]


@pytest.fixture(scope="module")
def ext():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_13511_amd import binding
    binding.lib()
    return binding


def trits(rows, cols, seed):
    """Half of the entries nonzero; no zero column."""
    rng = np.random.default_rng(seed)
    X = rng.choice(np.array([-1, 0, 0, 1], dtype=np.int8), size=(rows, cols))
    X[rng.integers(0, rows, size=cols), np.arange(cols)] = 1
    return X


def gram(X, w):
    X = X.astype(np.float64)
    G = X.T @ (w[:, None] * X)
    return G + oracle.RIDGE_REL * np.trace(G) / X.shape[1] * np.eye(X.shape[1])


def solve_eps(G):
    return 8.0 * G.shape[0] * np.linalg.cond(G) * 2.0 ** -53


@pytest.mark.parametrize("m,n,bb", NARROW + WIDE)
def test_vstep_edges(ext, m, n, bb):
    print(f"[edges] vstep {m}x{n} bb={bb}", flush=True)
    R, U, tau = synth.small("t4_rowscale", m, n, 7), trits(m, bb, m + bb), 0.7
    R64 = R.astype(np.float64)
    _, Y_ref = oracle.vstep(R64, U, tau)
    V, Y = ext.step_vstep(cuda(R), cuda(U), tau)
    V, Y = host(V), host(Y)
    G = gram(U, np.ones(m))
    dP = 2.0 ** -30 * np.abs(U).astype(np.float64).sum(axis=0)[:, None] * np.linalg.norm(R64, axis=0)[None, :]
    bound = np.abs(np.linalg.inv(G)) @ dP + 2.0 * solve_eps(G) * np.max(np.abs(Y_ref))
    assert np.all(np.abs(Y - Y_ref) <= bound)
    cols_parity(V, Y.T, tau, "V")


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("m,n,bb", NARROW + WIDE)
def test_ustep_edges(ext, m, n, bb, weighted):
    print(f"[edges] ustep {m}x{n} bb={bb} w={weighted}", flush=True)
    R, V, tau = synth.small("t4_rowscale", m, n, 8), trits(n, bb, n + bb), 0.7
    R64 = R.astype(np.float64)
    h = synth.small_importance(n, 8) if weighted else None
    w = oracle.normalized_weights(h, n)
    _, Q_ref, _ = oracle.ustep(R64, V, w, tau)
    U, Q, Z = ext.step_ustep(cuda(R), cuda(V), tau, h=cuda(h) if weighted else None)
    U, Q, Z = host(U), host(Q), host(Z)
    rmax = np.max(np.abs(R64 * w[None, :]), axis=1)
    assert np.all(np.abs(Q - Q_ref) <= 2.0 ** -29 * np.abs(V).astype(np.float64).sum(axis=0)[None, :] * rmax[:, None])
    G = gram(V, w)
    Z_chk = np.linalg.solve(G, Q.T).T
    bound = 2.0 * solve_eps(G) * np.max(np.abs(Z_chk))
    if weighted:
        Va = np.abs(V).astype(np.float64)
        bound = bound + 2.0 * np.abs(Z_chk) @ (2.0 ** -42 * np.max(w) * Va.T @ Va) @ np.abs(np.linalg.inv(G))
    assert np.all(np.abs(Z - Z_chk) <= bound)
    cols_parity(U, Z, tau, "U")


@pytest.mark.parametrize("m,n,bb", WIDE)
def test_wide_deflate_edges(ext, m, n, bb):
    print(f"[edges] deflate {m}x{n} bb={bb}", flush=True)
    R, U, V = synth.small("t4_rowscale", m, n, 9), trits(m, bb, m), trits(n, bb, n)
    d = np.random.default_rng(bb).standard_normal(bb).astype(np.float32).astype(np.float64)
    ref = oracle.deflate(R.astype(np.float64), U, V, d)
    Rt = cuda(R)
    col, fro = ext.step_deflate(Rt, cuda(U), cuda(V), cuda(d))
    Rg = host(Rt).astype(np.float64)
    scale = np.abs(R) + (np.abs(U).astype(np.float64) * np.abs(d)[None, :]) @ np.abs(V).astype(np.float64).T
    assert np.all(np.abs(Rg - ref) <= 2e-6 * ((bb + 63) // 64) * scale)
    np.testing.assert_allclose(host(col), np.sum(Rg * Rg, axis=0), rtol=1e-12)
    np.testing.assert_allclose(host(fro)[0], np.sum(Rg * Rg), rtol=1e-12)
