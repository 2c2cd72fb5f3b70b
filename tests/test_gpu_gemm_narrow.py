"""Tiled products whose right operand has one to three columns (fewer than a
thread loads at once), over two to five full slices of 16 with and without a
last partial one, against the oracle (tolerances as in test_gpu_gemm_edges.py);
and their time: they run the same pipeline as those of a few more columns, which
are the same tiles, so they may not take much longer."""
import numpy as np
import pytest

import synth
from helpers import rel, to_dev, to_host
from oracle import fd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import paper_1602_01636_amd as api
    api.lib()
    return api


@pytest.mark.parametrize("n2", [31, 32, 33, 47, 48, 64, 65, 80, 95])
@pytest.mark.parametrize("n1", [1, 2, 3])
def test_narrow(api, n1, n2, rng, monkeypatch):
    monkeypatch.setenv("IGAFD_FD_GEMM", "1")
    prob = synth.uniform_problem(2, [n1 + 1, n2 + 1], 1)
    F = fd.setup(prob)
    with api.igafd_setup_precond(prob) as ctx:
        assert list(ctx.n[:2]) == [n1, n2]
        r = rng.standard_normal(ctx.N)
        ref = fd.fd_apply(F, r)
        for prec, tol in (("fp64", 1e-11), ("fp32", 1e-4), ("bf16", 5e-2), ("bf16x3", 6e-4)):
            s = to_dev(np.full(ctx.N, np.nan))
            api.igafd_apply_precond(ctx, prec, to_dev(r), s)
            assert rel(to_host(s), ref) < tol, prec


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16", "bf16x3"])
def test_narrow_takes_no_longer_than_wider(api, prec):
    import torch

    def us(n1):  # one apply, the best of ten runs of forty
        with api.igafd_setup_precond(synth.uniform_problem(2, [n1, 1000], 2)) as ctx:
            r, s = (torch.ones(ctx.N, dtype=torch.float64, device="cuda") for _ in range(2))
            best = np.inf
            for _ in range(11):
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                a.record()
                for _ in range(40):
                    api.igafd_apply_precond(ctx, prec, r, s)
                b.record()
                b.synchronize()
                best = min(best, a.elapsed_time(b) * 1e3 / 40)
            return best

    narrow, wider = us(3), us(5)
    assert narrow < 1.25 * wider, (narrow, wider)


@pytest.mark.parametrize("E", [2, 3, 4, 5, 9])
def test_narrow_in_a_pair(api, E, monkeypatch):
    """The L-shaped domain's two subdomains, h x (2h + 1) and (2h + 1) x h with
    h = E - 1, share their launches: a narrow product beside one that is not."""
    from oracle import multipatch as mp
    monkeypatch.setenv("IGAFD_FD_GEMM", "1")
    knots = synth.uniform_knots(E, 1)
    L = mp.LShape(knots, 1)
    S = mp.Schwarz(L)
    pos, n = L.square_index()
    r = np.zeros(n * n)
    r[pos] = synth.random_vector(L.N, 5)
    ref = S.ias(r[pos])
    with api.igafd_lshape_setup(knots, 1) as ctx:
        for prec, tol in (("fp64", 1e-11), ("fp32", 1e-4), ("bf16", 5e-2), ("bf16x3", 6e-4)):
            s = to_dev(np.full(n * n, np.nan))
            api.igafd_apply_precond(ctx, prec, to_dev(r), s)
            assert rel(to_host(s)[pos], ref) < tol, prec
