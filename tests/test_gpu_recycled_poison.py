"""Contexts set up in recycled memory full of NaN give bitwise the results of a
context in fresh memory: element-order and across-element assembly, 2D and 3D,
scaling, ADI, in blocks of exactly the requested size and in larger ones.  The
problems are large enough (>= 1 MiB a buffer) that workspace, padded vectors,
band, features and scaling all come from the block cache; that they did is
checked: none of them is left in the cache."""
import ctypes as C

import numpy as np
import pytest

import synth
from helpers import to_dev, to_host

pytestmark = pytest.mark.gpu

W = synth.warped_geometry(1)
K = synth.sincos_coefficient()
CASES = {  # problem, features, then what runs beside the solves
    "3d": (synth.uniform_problem(3, [52, 53, 54], 2, geometry=W, coefficient=K), False, ""),
    "3d_features": (synth.uniform_problem(3, [52, 53, 54], 2, geometry=W, coefficient=K), True, ""),
    "3d_scaled": (synth.uniform_problem(3, [52, 53, 54], 2, geometry=W, coefficient=K), True, "scaled"),
    "3d_adi": (synth.uniform_problem(3, [52, 53, 54], 2, geometry={"kind": "ring"}), False, "adi"),
    "2d": (synth.uniform_problem(2, [410, 390], 3, geometry={"kind": "ring"}), False, ""),
    "2d_features": (synth.uniform_problem(2, [410, 390], 3, geometry={"kind": "ring"}), True, ""),
}


@pytest.fixture(scope="module")
def api():
    import paper_1602_01636_amd as api
    api.lib()
    return api


def _results(api, prob, features, extra, poisoned=()):
    import torch
    with api.igafd_setup(prob, features=features) as ctx:
        out = {}
        b = torch.empty(ctx.N, dtype=torch.float64, device="cuda")
        api.igafd_load_vector(ctx, synth.RHS_SINPROD, b)
        out["b"] = to_host(b)
        if extra == "scaled":
            api.igafd_set_scaling(ctx, to_dev(np.exp(0.1 * np.sin(np.arange(ctx.N)))))
        if extra == "adi":
            api.igafd_set_adi_greedy(ctx, 0.3)
        for prec in ("fp64",) if extra == "adi" else ("fp64", "bf16", "bf16x3"):
            u = torch.empty_like(b)
            api.igafd_solve(ctx, b, u, precision=prec, use_scaling=extra == "scaled")
            out["u " + prec] = to_host(u)
        if features:
            f = torch.empty(8 * ctx.N, dtype=torch.float32, device="cuda")
            api.igafd_features(ctx, f)
            out["features"] = to_host(f)
        taken = _alloc(api, [n for _, n in poisoned])  # a block still in the cache would be handed out here
        unused = {p.value for p, _ in poisoned} & {p.value for p in taken}
        _free(api, taken)
        return out, unused, ctx.N, ctx.band_bytes


def _alloc(api, sizes):
    alloc = api.lib()._ZN5igafd11block_allocEPPvm
    alloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
    ptrs = [C.c_void_p() for _ in sizes]
    for p, n in zip(ptrs, sizes):
        assert alloc(C.byref(p), n) == 0
    return ptrs


def _free(api, ptrs):
    free = api.lib()._ZN5igafd10block_freeEPvb
    free.argtypes, free.restype = [C.c_void_p, C.c_bool], None
    for p in ptrs:
        free(p, True)


def _poison(api, sizes):
    """Puts blocks of these sizes, all NaN, into the cache: (address, size)."""
    hip = C.CDLL("libamdhip64.so.7") if "libamdhip64.so.7" in open("/proc/self/maps").read() else C.CDLL("libamdhip64.so")
    ptrs = _alloc(api, sizes)
    for p, n in zip(ptrs, sizes):
        assert hip.hipMemset(p, C.c_int(0xFF), C.c_size_t(n)) == 0
    assert hip.hipDeviceSynchronize() == 0
    _free(api, ptrs)
    return list(zip(ptrs, sizes))


@pytest.mark.parametrize("name", list(CASES))
def test_poisoned_blocks(api, name):
    prob, features, extra = CASES[name]
    api.igafd_release_cached()
    want, _, N, band = _results(api, prob, features, extra)
    assert all(np.isfinite(v).all() for v in want.values())
    dim, p = prob["dim"], prob["degree"]
    w = 2 * p + 1
    Ns = band // 8 // ((w ** dim + 1) // 2)
    sizes = [band, 6 * 8 * ((N + 31) // 32 * 32), 8 * Ns, 8 * Ns]
    if features:
        sizes.append(32 * N)
    if extra == "scaled":
        sizes.append(8 * N)
    assert min(sizes) >= 1 << 20
    for slack in (1.0, 1.05):
        api.igafd_release_cached()
        poisoned = _poison(api, [int(slack * n) for n in sizes])
        got, unused, _, _ = _results(api, prob, features, extra, poisoned)
        assert not unused, (slack, sizes)
        for k in want:
            assert np.array_equal(got[k], want[k]), (k, slack)
    api.igafd_release_cached()
