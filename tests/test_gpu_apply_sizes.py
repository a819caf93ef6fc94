"""Inference at the sizes where its loads and segments have edges: packed rows
of any byte length at any byte address, matrices shorter than one load window,
and one vector past the length that a workgroup holds at once (more than
10240 components: segments of 16384, up to 65536, with the intermediate
rounded to fp32; fp32 sums past 65536).

The packed matrices lie in buffers whose other bytes are all ones (trit code
11, i.e. -1), so a byte taken from past a row or a matrix shows in the result.
Tolerances.  As derived in test_gpu_apply.py, one vector is exact integer sums
between two fixed-point conversions, more are fp32 sums of exact products.  One
long vector is converted without loss and summed exactly by groups of 38 binades,
added in fp64, or summed in fp64 where its side is small (n + k + 4 roundings of
2^-53 of the absolute sum); t and y are rounded to fp32 (u |B| |t| and u |y|).  No bound of
it names the largest entry.
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def pack(X):
    rows, cols = X.shape
    code = np.where(X == 0, 0, np.where(X > 0, 1, 3)).astype(np.uint8)
    code = np.concatenate([code, np.zeros((rows, (-cols) % 4), np.uint8)], axis=1).reshape(rows, -1, 4)
    return (code[:, :, 0] | (code[:, :, 1] << 2) | (code[:, :, 2] << 4) | (code[:, :, 3] << 6)).astype(np.uint8)


def place(P, offset):
    """P on the GPU at a byte offset inside a buffer of ones."""
    buf = torch.full((P.size + offset + 64,), 0xFF, dtype=torch.uint8, device="cuda")
    view = buf[offset:offset + P.size].view(P.shape)
    view.copy_(torch.from_numpy(P))
    return view


def check(m, n, k, nb, offset, scale=None):
    from paper_2607_13511_amd import binding
    rng = np.random.default_rng([m, n, k, nb, offset])
    B = rng.integers(-1, 2, size=(m, k)).astype(np.int8)
    C = rng.integers(-1, 2, size=(k, n)).astype(np.int8)
    D = rng.standard_normal(k).astype(np.float32).astype(np.float64)
    X = rng.standard_normal((nb, n)).astype(np.float32).astype(np.float64)
    if scale is not None:
        X = (X * scale(rng, X.shape)).astype(np.float32).astype(np.float64)
    Y = binding.apply(place(pack(B), offset), place(pack(C), offset), torch.from_numpy(D.astype(np.float32)).cuda(),
                      m, n, torch.from_numpy(X.astype(np.float32)).cuda()).cpu().numpy().astype(np.float64)
    ref = oracle.apply(B, C, D, X)
    Bf, Cf = np.abs(B).astype(np.float64), np.abs(C).astype(np.float64)
    if nb == 1:
        mx, sx, md = np.max(np.abs(X)), np.sum(np.abs(X)), np.max(np.abs(D))
        if max(n, k) > 65536:
            bound = (n + k + 4) * U * (Bf @ (np.abs(D) * (Cf @ np.abs(X[0]))))
        elif max(n, k) > 10240:
            bound = long_bound(B, C, D, X[0], ref)
        else:
            q = Bf @ (np.abs(D) * Cf.sum(axis=1)) * mx + Bf.sum(axis=1) * md * sx
            # twice the conversions (fp64 roundings); 1 + 2^-20: second-order terms
            bound = U * np.abs(ref[0]) * (1.0 + 2.0 ** -20) + 2.0 * 2.0 ** -46 * q
        assert np.all(np.abs(Y[0] - ref[0]) <= bound)
    else:
        bound = ((n + k + 4) * U * (Bf @ (np.abs(D)[:, None] * (Cf @ np.abs(X).T)))).T
        assert np.all(np.abs(Y - ref) <= bound)


def long_bound(B, C, D, x, ref):
    """Of one long vector; 1 + 2^-20: second-order terms."""
    (m, k), n = B.shape, C.shape[1]
    Bf, Cf = np.abs(B).astype(np.float64), np.abs(C).astype(np.float64)
    t = D * (C.astype(np.float64) @ x)
    return (U * (np.abs(ref[0]) + Bf @ np.abs(t)) * (1.0 + 2.0 ** -20)
            + (n + k + 4) * 2.0 ** -53 * (Bf @ (np.abs(D) * (Cf @ np.abs(x)))))


@pytest.mark.parametrize("nb", [1, 3, 8])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (1, 61, 3), (3, 5, 70), (2, 28, 31), (17, 65, 63), (16, 254, 513),
                                   (65, 1021, 259), (257, 130, 1030)])
def test_row_lengths(m, n, k, nb):
    check(m, n, k, nb, 0)


@pytest.mark.parametrize("nb", [1, 2, 6])
@pytest.mark.parametrize("offset", [1, 4, 8, 15])
def test_byte_addresses(offset, nb):
    check(33, 256, 320, nb, offset)   # rows of 64 and 80 bytes: only the base is off
    check(19, 250, 330, nb, offset)


@pytest.mark.parametrize("m,n,k", [(40, 10241, 33), (16, 33, 20481), (33, 20480, 48), (17, 30723, 10245),
                                   (5, 65536, 7), (3, 9, 65535)])
def test_one_long_vector(m, n, k):
    check(m, n, k, 1, 0)
    check(m, n, k, 1, 1, lambda rng, shape: np.exp2(rng.integers(-20, 1, size=shape)))


@pytest.mark.parametrize("m,n,k", [(4096, 10241, 20), (4097, 10241, 20), (12289, 10300, 61), (32768, 10241, 16),
                                   (32769, 10241, 16), (9, 16640, 4100), (4113, 33, 16641)])
def test_one_long_vector_tiles(m, n, k):
    """Workgroups of one, two, more and the most row tiles, also over several
    segments, on each side; rows off every load width, at word addresses and off them."""
    for offset in (0, 4, 6):
        check(m, n, k, 1, offset)


@pytest.mark.parametrize("gap", [20, 24, 30, 38, 39, 40, 60, 120])
@pytest.mark.parametrize("side", ["x", "t"])
def test_long_vector_small_entries(side, gap):
    """One entry 2^gap above the others, where half of the rows have no trit:
    their results keep their own accuracy."""
    from paper_2607_13511_amd import binding
    print(f"[apply] {side} gap {gap}", flush=True)
    m, n, k = (35, 12005, 50) if side == "x" else (50, 37, 12005)
    rng = np.random.default_rng([gap, n])
    B = rng.integers(-1, 2, size=(m, k)).astype(np.int8)
    C = rng.integers(-1, 2, size=(k, n)).astype(np.int8)
    D = rng.standard_normal(k).astype(np.float32).astype(np.float64)
    x = rng.standard_normal(n).astype(np.float32).astype(np.float64)
    at = 7777
    if side == "x":
        x[at] = 2.0 ** gap
        C[::2, at] = 0
        B[::3, 1::2] = 0     # these outputs see only rows of C without the large entry
    else:
        D[at] *= 2.0 ** gap
        C[at, 3] = 1
        B[::2, at] = 0
    if gap == 120:           # the others denormal in fp32
        x = (x * 2.0 ** -135).astype(np.float32).astype(np.float64)
        if side == "x":
            D = D * 2.0 ** 80
    Y = binding.apply(place(pack(B), 3), place(pack(C), 3), torch.from_numpy(D.astype(np.float32)).cuda(), m, n,
                      torch.from_numpy(x.astype(np.float32)[None, :]).cuda()).cpu().numpy().astype(np.float64)
    ref = oracle.apply(B, C, D, x[None, :])
    bound = long_bound(B, C, D, x, ref) + 2.0 ** -149 * (1.0 + np.abs(B).sum(axis=1))   # denormal t and y
    assert np.all(np.abs(Y[0] - ref[0]) <= bound)


@pytest.mark.parametrize("m,n,k", [(6, 65537, 12), (9, 20, 65537)])
def test_one_vector_past_the_long_path(m, n, k):
    check(m, n, k, 1, 0)
    check(m, n, k, 1, 1)


def test_several_long_vectors():
    check(6, 65537, 12, 3, 0)   # the slices, at any length


def test_long_vector_spread():
    """Entries over 120 binades: several passes of k_gemv_long on either side."""
    check(35, 12005, 50, 1, 0, lambda rng, shape: np.exp2(rng.integers(-120, 1, size=shape)))
    check(40, 17000, 700, 1, 4, lambda rng, shape: np.exp2(rng.integers(-100, 1, size=shape) * (rng.random(shape) < 0.01)))


def test_long_vector_nonfinite():
    from paper_2607_13511_amd import binding
    C = np.ones((4, 12000), np.int8)
    B = np.ones((3, 4), np.int8)
    for bad in (np.nan, np.inf):
        X = np.ones((1, 12000), np.float32)
        X[0, 11999] = bad
        Y = binding.apply(place(pack(B), 0), place(pack(C), 0), torch.ones(4, device="cuda"), 3, 12000,
                          torch.from_numpy(X).cuda())
        assert torch.isnan(Y).all()


def test_small_side_nonfinite():
    from paper_2607_13511_amd import binding
    C, B = np.ones((12000, 20), np.int8), np.ones((3, 12000), np.int8)
    for bad in (np.nan, np.inf):
        X = np.ones((1, 20), np.float32)
        X[0, 19] = bad
        Y = binding.apply(place(pack(B), 0), place(pack(C), 0), torch.ones(12000, device="cuda"), 3, 20,
                          torch.from_numpy(X).cuda())
        assert torch.isnan(Y).all()
