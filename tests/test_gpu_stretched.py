"""Rotated boxes whose edges differ in length by orders of magnitude, in FP64: the error of the
on-the-fly factors stays a few roundings, as from differences of neighbouring vertices, and does not
grow with the aspect ratio.  Every kernel that recomputes the factors, against factors evaluated in
80 bits."""
import numpy as np
import pytest

import oracle
from gpu_util import U64, check_bound

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ax():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2504_07042_amd as ax
    ax.lib()
    return ax


def _boxes(n, axis, aspect, seed):
    """n rotated boxes near the origin, `aspect` times shorter along `axis` than along the others."""
    rng = np.random.default_rng(seed)
    corners = np.array([[a, b, c] for c in (0, 1) for b in (0, 1) for a in (0, 1)], float) - 0.5
    size = np.ones(3)
    size[axis] = 1.0 / aspect
    q = [np.linalg.qr(rng.normal(size=(3, 3)))[0] for _ in range(n)]
    q = [m if np.linalg.det(m) > 0 else -m for m in q]
    return np.stack([(corners * size) @ m.T + 0.3 * rng.uniform(-1, 1, 3) for m in q])


def _factors80(verts, xi, w):
    """G [E][6][N1^3] of the given vertices, every step in 80 bits."""
    T = np.longdouble
    x = (verts.astype(T) / 8).reshape(-1, 2, 2, 2, 3)             # E t s r q
    f = np.stack([1 - xi.astype(T), 1 + xi.astype(T)])            # 2 n
    g = np.stack([-np.ones(len(xi), T), np.ones(len(xi), T)])
    # differences along the derivative's direction first, then the blends
    J = [np.einsum("ck,bj,ai,ecbaq->ekjiq", *((g if d == 2 else f), (g if d == 1 else f), (g if d == 0 else f)),
                   x) for d in range(3)]
    C = [np.cross(J[1], J[2]), np.cross(J[2], J[0]), np.cross(J[0], J[1])]
    W = (w.astype(T)[:, None, None] * w.astype(T)[:, None] * w.astype(T)) / (J[0] * C[0]).sum(-1)
    G = [(C[a] * C[b]).sum(-1) * W for a, b in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))]
    return np.stack(G, 1).reshape(len(verts), 6, -1).astype(np.float64)


def _bound(N):
    """In units of the envelope |D|^T S |D| |X|, S_ab = sqrt(G_aa G_bb): 2 N1 + 8 roundings of the two
    contractions and 3-term sums, here and in the oracle, and 48 of a factor: an edge 1, its sum and
    blends 5, products of three columns with their sums 3 x 3 + 2, the polynomial in t 4 and the adjugate
    4, each of these twice where the entry is a product of two; scale and reciprocal 6."""
    return (2 * (2 * (N + 1) + 8) + 48) * U64


def _case(N, axis, aspect, E=21):
    from paper_2504_07042_amd import Basis
    b = Basis(N)   # the kernels' own tables (the oracle's differ from them by up to 10^-14 at N = 15)
    D = np.asarray(b.D).reshape(N + 1, N + 1)
    V = _boxes(E, axis, aspect, seed=10 * N + axis)
    G = _factors80(V, np.asarray(b.xi), np.asarray(b.w))
    X = np.random.default_rng(N).uniform(-1, 1, (2, E, (N + 1) ** 3))
    S = np.sqrt(G[:, [0, 0, 0, 3, 3, 5]] * G[:, [0, 3, 5, 3, 5, 5]])
    return V, X, oracle.ax_local(D, G, X), oracle.ax_envelope(D, S, X)


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("aspect", [1.0, 1e4])
@pytest.mark.parametrize("N", [1, 2, 3, 5, 7, 8, 9, 11, 14, 15])
def test_single_mesh(ax, N, aspect, axis):
    from paper_2504_07042_amd import autotune
    V, X, Yref, env = _case(N, axis, aspect)
    b, v, x = ax.Basis(N), _dev(V), _dev(X)
    K = ax.AX_TUNE_TRILINEAR
    saved = autotune.tune_get(N, K, ax.AX_FP64)
    try:
        for kernel in (ax.AX_KERNEL_TILE, ax.AX_KERNEL_ITEM):
            autotune.tune_set(N, K, ax.AX_FP64, kernel=kernel)
            for cols in (1, 2):
                Y = ax.ax_local(x[:cols].contiguous(), v, b).cpu().numpy()
                check_bound(Y, Yref[:cols], env[:cols], _bound(N), tag=f"boxes {aspect:g} axis {axis} N={N} {kernel}")
    finally:
        autotune.tune_set(N, K, ax.AX_FP64, **{k: saved[k] for k in autotune.KNOBS})
    Y = ax.ax_local_partial(x, v, ax.geom_lambda(v, b), b).cpu().numpy()
    check_bound(Y, Yref, env, _bound(N), tag=f"boxes {aspect:g} axis {axis} N={N} partial")


@pytest.mark.parametrize("shape", [(0, 0, 0), (0, 1, 0), (1, 0, 0), (1, 0, 1)])
def test_batched(ax, shape):
    """Per-item shapes 0 and 1, the tile kernel over the work list and over mesh slices."""
    import torch
    from paper_2504_07042_amd import autotune
    tile, item_alt, tile_alt = shape
    orders = range(1, 10)
    cases = [_case(N, N % 3, 1e4) for N in orders]
    K = ax.AX_TUNE_BATCHED
    saved = {N: autotune.tune_get(N, K, ax.AX_FP64) for N in orders}
    try:
        for N in orders:
            autotune.tune_set(N, K, ax.AX_FP64, kernel=ax.AX_KERNEL_TILE if tile else ax.AX_KERNEL_ITEM,
                              item_alt=item_alt, tile_alt=tile_alt)
        X = [_dev(c[1]) for c in cases]
        Y = [torch.empty_like(x) for x in X]
        ax.BatchedAxLocal([(_dev(c[0]), ax.Basis(N)) for N, c in zip(orders, cases)], X, Y, ax.AX_FP64).launch()
        torch.cuda.synchronize()
    finally:
        for N, s in saved.items():
            autotune.tune_set(N, K, ax.AX_FP64, **{k: s[k] for k in autotune.KNOBS})
    for N, c, y in zip(orders, cases, Y):
        check_bound(y.cpu().numpy(), c[2], c[3], _bound(N), tag=f"batched boxes {shape} N={N}")
