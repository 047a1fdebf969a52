"""Gram-Schmidt kernels themselves: projections, update, norm, and the projections that the update leaves for a second pass.

Through the Arnoldi driver a wrong second projection stays unseen (it corrects a vector that is orthogonal to rounding
already, and what it takes out goes into the Hessenberg matrix), so the launchers are called directly, with a
basis that is not orthogonal and coefficients that are not the projections, so that every digit counts.  Numbers of
vectors on both sides of the instances (4, 8, .. 24, 32, 40, 48), lengths from one value to several rounds of
all blocks (512 of 256 values, or of pairs), odd and even.

Tolerances: a sum over n terms is made of at most n / 2^16 + 32 additions in a row (per thread, wave, block, blocks),
each with a relative error of u = 2^-53 of the terms' absolute sum; 64 u covers them for n below 2^21.  An
updated value is nv products and sums: (nv + 2) u of their absolute sum.  References in extended precision.
"""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = 2.0**-53
LENGTHS = [1, 2, 255, 257, 1001, 262145, 300002]


def functions():
    import paper_1704_08521_amd as lk
    lib = lk._lib.load()
    p, i, l, z = C.c_void_p, C.c_int, C.c_long, C.c_size_t
    sig = {"dot": ("_ZN2lk13launch_gs_dotEPKdlibS1_mPdS2_S2_P12ihipStream_t", [p, l, i, C.c_bool, p, z, p, p, p, p]),
           "update": ("_ZN2lk16launch_gs_updateEPKdliS1_PdmS2_P12ihipStream_t", [p, l, i, p, p, z, p, p]),
           "fused": ("_ZN2lk20launch_gs_update_dotEPKdliS1_PdmS2_S2_S2_S2_P12ihipStream_t",
                     [p, l, i, p, p, z, p, p, p, p, p]),
           "parts": ("_ZN2lk15gs_update_partsEm", [z]), "fused_parts": ("_ZN2lk19gs_update_dot_partsEmi", [z, i])}
    out = {}
    for k, (name, args) in sig.items():
        out[k] = getattr(lib, name)
        out[k].argtypes, out[k].restype = args, i
    return out


@pytest.mark.parametrize("nv", [1, 4, 5, 8, 9, 16, 20, 24, 25, 32, 33, 40, 41, 48, 49, 64])
def test_projections_and_update(nv):
    import torch
    f = functions()
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    ptr = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    for n in LENGTHS:
        print(f"[case] nv = {nv}, n = {n}", flush=True)
        ld = (n + 63) // 64 * 64
        rng = np.random.default_rng(1000 * nv + n)
        V = np.full((nv, ld), np.nan)  # what lies between the vectors is not read
        V[:, :n] = rng.standard_normal((nv, n)) / np.sqrt(n)
        w, h = rng.standard_normal(n), rng.standard_normal(nv)
        v = V[:, :n].astype(np.longdouble)
        dV, dh = dev(V), dev(h)
        scratch, out = torch.zeros(512 * 32, dtype=torch.float64, device="cuda"), torch.full((nv + 2,), -1.0, dtype=torch.float64, device="cuda")
        # projections, with the norm as one more
        dw = dev(w)
        assert f["dot"](ptr(dV), ld, nv, True, ptr(dw), n, ptr(scratch), ptr(out), None, stream) == 0
        got = out.cpu().numpy()
        rows = np.vstack([v, w.astype(np.longdouble)])
        assert np.all(np.abs(got[:-1] - rows @ w) <= 64 * U * (np.abs(rows) @ np.abs(w)))
        assert got[-1] == -1.0
        # the update, alone and with the projections of its result
        ref = w - h @ v
        bound = (nv + 2) * U * (np.abs(w) + np.abs(h) @ np.abs(v))
        for kind in ("update",) + (("fused",) if nv <= 48 else ()):
            dw, out = dev(np.append(w, 7.0)), torch.full((nv + 1,), -1.0, dtype=torch.float64, device="cuda")
            parts = f["parts"](n) if kind == "update" else f["fused_parts"](n, nv)
            assert 1 <= parts <= 1024
            sums = torch.full((parts + 1,), -1.0, dtype=torch.float64, device="cuda")
            if kind == "update":
                rc = f["update"](ptr(dV), ld, nv, ptr(dh), ptr(dw), n, ptr(sums), stream)
            else:
                rc = f["fused"](ptr(dV), ld, nv, ptr(dh), ptr(dw), n, ptr(sums), ptr(scratch), ptr(out), None, stream)
            assert rc == 0
            x, s = dw.cpu().numpy(), sums.cpu().numpy()
            assert x[n] == 7.0 and s[parts] == -1.0
            x = x[:n]
            assert np.all(np.abs(x - ref) <= bound), kind
            assert abs(np.sum(s[:parts].astype(np.longdouble)) - np.sum(x.astype(np.longdouble)**2)) <= 64 * U * np.sum(x * x)
            if kind == "fused":
                got = out.cpu().numpy()
                assert np.all(np.abs(got[:nv] - v @ x) <= 64 * U * (np.abs(v) @ np.abs(x)))
                assert got[nv] == -1.0
