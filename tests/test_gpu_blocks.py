"""Recycled device blocks: contexts set up in memory that earlier contexts left
behind (of other problems, precisions and threads) give bitwise the results of
the first context, also from several host threads on their own streams; equal
and unequal directions (shared and separate eigendecompositions)."""
import threading

import numpy as np
import pytest

import synth
from helpers import to_host

pytestmark = pytest.mark.gpu


def _problems():
    u = synth.uniform_knots
    return [
        synth.make_problem(3, 3, [u(24, 3)] * 3, synth.warped_geometry(1), synth.sincos_coefficient()),
        synth.make_problem(3, 3, [u(24, 3), u(23, 3), synth.jittered_knots(24, 3, 5)], {"kind": "ring"}),
        synth.make_problem(3, 4, [u(17, 4), u(17, 4), u(18, 4)], synth.warped_geometry(2)),
    ]


def _run(api, torch, prob):
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        with api.igafd_setup(prob, features=True) as ctx:
            b = torch.empty(ctx.N, dtype=torch.float64, device="cuda")
            u = torch.empty_like(b)
            feat = torch.empty(8 * ctx.N, dtype=torch.float32, device="cuda")
            api.igafd_load_vector(ctx, synth.RHS_SINPROD, b)
            api.igafd_features(ctx, feat)
            for prec in ("bf16", "fp64"):  # leaves other bit patterns in the workspace
                api.igafd_solve(ctx, b, u, precision=prec)
            stream.synchronize()
            return [to_host(t) for t in (b, u, feat)]


def test_recycled_blocks_are_bitwise_neutral():
    import torch

    import paper_1602_01636_amd as api
    api.lib()
    probs = _problems()
    ref = [_run(api, torch, p) for p in probs]
    for r in ref:
        assert all(np.isfinite(v).all() for v in r)
    for k in (1, 0, 2, 1, 0):
        for got, want in zip(_run(api, torch, probs[k]), ref[k]):
            assert np.array_equal(got, want), k
    errors = []

    def work(first):
        try:
            for k in range(4):
                i = (first + k) % len(probs)
                for got, want in zip(_run(api, torch, probs[i]), ref[i]):
                    assert np.array_equal(got, want), (first, i)
        except BaseException as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
