"""GPU parity of the tiled products' slice pipeline at its edges: fewer than one
and exactly one, two and three slices of 16, with and without a last partial
one; one to three columns (fewer than a thread loads at once); one column,
row or point past a tile; both operand forms (direction 1 and the others), every
precision, plain and scaled.  Tolerances as for the applies of
test_gpu_parity.py and test_gpu_cube.py.
"""
import numpy as np
import pytest

import synth
from helpers import rel, to_dev, to_host
from oracle import fd

pytestmark = pytest.mark.gpu

CASES = [  # elements per direction (p = 1: unknowns one fewer), so unknowns per direction:
    (2, 3, 4), (3, 2, 18), (4, 17, 16),          # 1 2 3; 2 1 17; 3 16 15
    (5, 33, 34), (6, 49, 48), (17, 18, 66),      # 4 32 33; 5 48 47; 16 17 65
    (66, 129, 7), (130, 5, 65),                  # 65 128 6; 129 4 64
    (2, 200), (65, 33), (130, 131), (400, 3),    # 2D
]


@pytest.fixture(scope="module")
def api():
    import paper_1602_01636_amd as api
    api.lib()
    return api


@pytest.mark.parametrize("els", CASES, ids=["x".join(map(str, e)) for e in CASES])
def test_gemm_edges(api, els, rng, monkeypatch):
    monkeypatch.setenv("IGAFD_FD_GEMM", "1")
    prob = synth.uniform_problem(len(els), list(els), 1)
    F = fd.setup(prob)
    with api.igafd_setup(prob) as ctx:
        r = rng.standard_normal(ctx.N)
        S = np.exp(0.1 * rng.standard_normal(ctx.N))
        for scaled in (False, True):
            if scaled:
                api.igafd_set_scaling(ctx, to_dev(S))
            ref = S * fd.fd_apply(F, S * r) if scaled else fd.fd_apply(F, r)
            for prec, tol in (("fp64", 1e-11), ("fp32", 1e-4), ("bf16", 5e-2), ("bf16x3", 6e-4)):
                s = to_dev(np.full(ctx.N, np.nan))
                api.igafd_apply_precond(ctx, prec, to_dev(r), s)
                assert rel(to_host(s), ref) < tol, (prec, scaled)
