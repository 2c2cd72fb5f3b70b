"""GPU parity of the fused ADI sub-steps at the edges of their rule: blocks of
32 and of 16 lines, partial last blocks, lines shorter than the band and than a
thread's run, lines too long for LDS in each direction (unfused sub-steps), and a
last sub-step with more blocks than the partial sums hold.  One apply against the
oracle's closed form within max(1e-11, eps kappa) as for the full-size apply
(test_gpu_adi.py), and its dot product inside a CG solve through the true residual.
"""
import numpy as np
import pytest

import synth
from helpers import rel, to_dev, to_host
from oracle import adi, fd

pytestmark = pytest.mark.gpu

CASES = [  # elements per direction, degree
    ((33, 30, 31), 3),   # 32 lines a block, partial last blocks
    ((3, 2, 2), 5),      # lines of 4 to 6 points, fewer than a thread's run
    ((1, 2, 3), 2),      # a line of one point
    ((70, 131, 9), 3),   # 16 lines a block in direction 2's neighbours
    ((120, 110, 100), 2),
    ((460, 3, 2), 3),    # direction 1 too long for three vectors in LDS
    ((2, 700, 3), 3),    # direction 2 too long
    ((3, 2, 500), 3),    # direction 3 too long for two vectors
    ((40, 300, 300), 1),
    ((7, 200, 6), 6),
    ((300, 260, 2), 1),  # last sub-step: more blocks of lines than of 256 unknowns
]


@pytest.fixture(scope="module")
def api():
    import paper_1602_01636_amd as api
    api.lib()
    return api


@pytest.mark.parametrize("els,p", CASES, ids=["x".join(map(str, e)) + f"_p{p}" for e, p in CASES])
def test_adi_lines(api, els, p):
    prob = synth.uniform_problem(3, list(els), p)
    F = fd.setup(prob)
    w, _, _ = adi.parameters(F, 0.1)
    kappa = max(f["lam"].max() for f in F) / min(f["lam"].min() for f in F)
    with api.igafd_setup(prob) as ctx:
        J, _ = api.igafd_set_adi(ctx, 0.1)
        assert J == len(w)
        x = synth.random_vector(ctx.N, 11)
        s = to_dev(np.full(ctx.N, np.nan))
        for _ in range(2):
            api.igafd_apply_precond(ctx, "fp64", to_dev(x), s)
            assert rel(to_host(s), adi.closed_form(F, x, w)) < max(1e-11, 2.2e-16 * kappa)
        b = to_dev(x)
        u = to_dev(np.zeros(ctx.N))
        info = api.igafd_solve(ctx, b, u, rtol=1e-8)
        assert info["status"] == "OK" and info["true_relres"] <= 1e-8
