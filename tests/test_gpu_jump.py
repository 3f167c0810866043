"""GPU: levels that jump over many power-iteration steps at once, on every
kernel that refines a level, against the oracle's plain loop: the same step
counts, the vector and the eigenvalue at the FP64 bar.

Tolerances: those of the FP64 parity tests (tests/gpu_compare.py).  A jump's
rounding error is that of a few steps (its coefficients are positive and
every Chebyshev vector has at most the start's norm), so they apply as they
are."""
import numpy as np
import pytest

from gpu_compare import COS_TOL, LAM_RTOL, oracle_of, run_gpu, say
from paper_1412_0565_amd import graphs as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1412_0565_amd import cmg

    cmg.lib()


def _chunglu(n, seed):
    return G.chung_lu(n, 2.5, 8.0, float(np.sqrt(8.0 * n)), seed=seed, int_weights=True)


GRAPHS = {
    "cl20k": lambda: _chunglu(20000, 3),
    "cl3k": lambda: _chunglu(3000, 5),
    "path400": lambda: G.path(400),
    "grid60x40": lambda: G.grid2d(60, 40),
}


def _check(g, got, ref):
    lam, x, st, levels, _ = got
    ks = [L.k for L in levels]
    say(f"  steps {ks} oracle {[L.k for L in ref.levels]} lambda {lam!r} oracle {ref.lam!r}")
    assert ks == [L.k for L in ref.levels]
    cos = abs(float(x @ ref.y)) / (np.linalg.norm(x) * np.linalg.norm(ref.y))
    assert cos >= 1 - COS_TOL
    assert abs(lam - ref.lam) <= LAM_RTOL * ref.lam
    return ks


# the defaults (persistent, merge-path and register-row levels, CSR levels in
# one workgroup), one launch per step, only grid kernels, only the CSR
# traversal in one workgroup, only merge path
@pytest.mark.parametrize("opts", [{}, {"step_mode": 1, "block_rows": 1}, {"block_rows": 1}, {"block_regs": -1},
                                  {"spmv_variant": 2, "block_rows": 1}],
                         ids=["default", "step", "grid", "csr", "merge"])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_jumps_keep_step_counts(name, opts):
    g = GRAPHS[name]()
    say(f"[jump] {name} {opts}")
    ks = _check(g, run_gpu(g, **opts), oracle_of(g))
    if name != "path400":  # its levels are too short for a jump
        assert max(ks) >= 150


# a fixed count is jumped without a test; 130 leaves a jump of the least length
@pytest.mark.parametrize("k0", [130, 900])
@pytest.mark.parametrize("opts", [{}, {"block_rows": 1}], ids=["default", "grid"])
def test_jumps_on_a_fixed_schedule(k0, opts):
    g = GRAPHS["cl3k"]()
    kw = dict(fixed_k0=k0, fixed_beta=1.0)
    _check(g, run_gpu(g, **kw, **opts), oracle_of(g, **kw))


# the cap ends a level inside what would be a jump
@pytest.mark.parametrize("cap", [140, 300])
@pytest.mark.parametrize("opts", [{}, {"step_mode": 1, "block_rows": 1}], ids=["default", "step"])
def test_jumps_stop_at_the_cap(cap, opts):
    g = GRAPHS["cl3k"]()
    ks = _check(g, run_gpu(g, max_iters_per_level=cap, **opts), oracle_of(g, max_iters_per_level=cap))
    assert cap in ks
