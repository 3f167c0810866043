"""GPU: the kernels that keep a small level in one workgroup, at the edges of
their ranges, against the oracle: dense levels (tiles of 16), register rows
with weights that single precision cannot hold, small levels of several
eigenpairs, and their setup (integers and weights bit for bit).

Tolerances: those of the FP64 parity tests (tests/gpu_compare.py); a dense
level's blocks of 16 steps and the block's reciprocal square roots round as
often as the plain steps do, so they apply as they are."""
import numpy as np
import pytest

from gpu_compare import COS_TOL, LAM_RTOL, assert_hierarchy_equal, oracle_of, run_gpu, say
from paper_1412_0565_amd import graphs as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1412_0565_amd import cmg

    cmg.lib()


def _real(g):
    """g with a weight of its own, far from single precision, on every edge."""
    row = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    a, b = np.minimum(row, g.col), np.maximum(row, g.col)
    up = row < g.col
    w = 0.5 + ((a * 7919 + b * 104729) % 1009) / 1009.0
    return G.from_edges(g.n, row[up], g.col[up], w[up])


def _check(g):
    ref = oracle_of(g)
    lam, x, _, levels, _ = run_gpu(g)
    say(f"  steps {[L.k for L in levels]} oracle {[L.k for L in ref.levels]} lambda {lam!r} oracle {ref.lam!r}")
    assert [L.k for L in levels] == [L.k for L in ref.levels]
    assert abs(float(x @ ref.y)) / (np.linalg.norm(x) * np.linalg.norm(ref.y)) >= 1 - COS_TOL
    assert abs(lam - ref.lam) <= LAM_RTOL * ref.lam


# up to 64 vertices, up to 128 with short rows, up to 176 nearly full, one
# more than each; p is the edge probability
@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("n,p", [(26, 0.3), (32, 0.3), (33, 0.3), (48, 0.2), (49, 0.2), (64, 0.3), (65, 0.1),
                                 (96, 0.1), (97, 0.1), (128, 0.08), (129, 0.5), (143, 0.4), (144, 0.6), (145, 0.5),
                                 (176, 0.6), (177, 0.6)])
def test_dense_levels(n, p, real):
    g = G.erdos_renyi_connected(n, p, seed=n)
    say(f"[dense] n={g.n} nnz={g.row_ptr[-1]} real={real}")
    _check(_real(g) if real else g)


@pytest.mark.parametrize("n", [150, 600, 1500, 4000])
def test_register_rows_in_double_precision(n):
    _check(_real(G.rgg(n, 9.0, seed=n)))


# one row of threads more or less than a wavefront and than the workgroup
# (1025 vertices run one launch per step); full rows beyond the LDS
@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("name", ["grid32x2", "grid13x5", "grid31x33", "grid128x8", "grid41x25", "er1000"])
def test_block_levels(name, p):
    from oracle import oracle as O
    from paper_1412_0565_amd import cmg

    g = G.erdos_renyi_connected(1000, 0.04, seed=4) if name == "er1000" else G.grid2d(*map(int, name[4:].split("x")))
    ref = O.cmg_block(g, p)
    if ref.status == "E_ARG" and name == "er1000":
        pytest.skip("its coarsest level is too small for p columns")
    assert ref.status == "OK"
    with cmg.Fiedler(g.n, g.row_ptr, g.col, g.w) as F:
        lams, X, res, steps = F.solve_block(p)
    say(f"[block] {name} p={p} steps {steps} oracle {ref.k} lams {lams} oracle {ref.lams}")
    assert steps == ref.k
    for c in range(p):
        assert float(X[:, c] @ ref.X[:, c]) / (np.linalg.norm(X[:, c]) * np.linalg.norm(ref.X[:, c])) >= 1 - COS_TOL
        assert abs(lams[c] - ref.lams[c]) <= LAM_RTOL * ref.lams[c]
    assert np.allclose(X.T @ X, np.eye(p), atol=1e-11)


# shares of the merge path that a jump holds in registers, at hub rows that
# leave one share too large (5000 entries and 1800 of other rows against 6144) and at real weights
@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("hub", [0, 2000, 5000])
def test_held_merge_products(hub, real):
    g = G.chung_lu(20000, 2.5, 8.0, 400.0, seed=3, int_weights=True)
    row = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    up = row < g.col
    far = np.arange(1, g.n, max(1, g.n // hub))[:hub] if hub else np.arange(0)
    u, v = np.concatenate([row[up], np.zeros(len(far), int)]), np.concatenate([g.col[up], far])
    _, at = np.unique(u.astype(np.int64) * g.n + v, return_index=True)
    g = G.from_edges(g.n, u[at], v[at])
    g = _real(g) if real else g
    ref = oracle_of(g)
    lam, x, _, levels, _ = run_gpu(g, spmv_variant=2, block_rows=1)
    say(f"[merge] hub={hub} real={real} steps {[L.k for L in levels]} oracle {[L.k for L in ref.levels]}")
    assert [L.k for L in levels] == [L.k for L in ref.levels]
    assert max(L.k for L in levels) >= 130  # a jump
    assert abs(float(x @ ref.y)) / (np.linalg.norm(x) * np.linalg.norm(ref.y)) >= 1 - COS_TOL
    assert abs(lam - ref.lam) <= LAM_RTOL * ref.lam


# one slot tile or many (13312 slots), rows of a few entries or near the
# longest, members of one aggregate only
@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("name", ["path26", "cycle27", "grid8x4", "grid64x128", "rgg1300", "rgg8000", "er300", "er8000"])
def test_small_level_setup(name, real):
    g = {"path26": lambda: G.path(26), "cycle27": lambda: G.cycle(27), "grid8x4": lambda: G.grid2d(8, 4),
         "grid64x128": lambda: G.grid2d(64, 128), "rgg1300": lambda: G.rgg(1300, 10.0, seed=2),
         "rgg8000": lambda: G.rgg(8000, 11.0, seed=3), "er300": lambda: G.erdos_renyi_connected(300, 0.03, seed=4),
         "er8000": lambda: G.erdos_renyi_connected(8000, 0.00105, seed=5)}[name]()
    g = _real(g) if real else g
    _, _, _, levels, arrays = run_gpu(g)
    say(f"[setup] {name} real={real} {[(L.n, L.nnz) for L in levels]}")
    assert_hierarchy_equal(g, oracle_of(g), levels, arrays, exact_g=False)
