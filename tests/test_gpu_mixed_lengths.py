"""Compile-time mixed-radix passes over their whole table (7-smooth lengths 16
.. 1024 but 343 and 686), both precisions, against the FP64 oracle.

Per length n the grids (n, 3, n) -- X and Z at length n, 3 n lines, a ragged
last column block, a half-empty last line pair for odd n -- and (5, n, 4) -- Y
at length n with 3 valid columns in the only block.  Forward of a uniform field
and backward of an arbitrary half spectrum, STRIDE1 for even table positions
and [nz][ny][nxh] rows for odd ones.

Bounds on the relative L2 error: 1e-6 in FP32 (the bound of every FP32 test
here); in FP64 1e-14: at most 10 butterfly levels per axis over 3 axes, each
contributing below 1.5 ulp (2.2e-16).
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1905_02803_amd as pf  # noqa: E402

LENGTHS = [n for n in synth.smooth7(16, 1024) if n not in (343, 686)]


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("prec", [pf.PF_F32, pf.PF_F64], ids=["f32", "f64"])
@pytest.mark.parametrize("part", range(8))
def test_every_length_in_every_role(prec, part):
    f64 = prec == pf.PF_F64
    tol = 1e-14 if f64 else 1e-6
    for i, n in list(enumerate(LENGTHS))[part::8]:
        stride1 = (i // 8) % 2
        for nx, ny, nz in ((n, 3, n), (5, n, 4)):
            print(f"case mixed-radix {nx}x{ny}x{nz} f64={f64} stride1={stride1}", flush=True)
            u = synth.uniform(n, (nz, ny, nx)).astype(np.float64 if f64 else np.float32)
            V = synth.complex_half(n + 1, (nz, ny, nx // 2 + 1)).astype(np.complex128 if f64 else np.complex64)
            to_layout = oracle.to_stride1 if stride1 else (lambda a: a)
            with pf.Plan(nx, ny, nz, pf.Layout(stride1=stride1, precision=prec)) as plan:
                U = plan.ftran(torch.from_numpy(u).cuda())
                b = plan.btran(torch.from_numpy(np.ascontiguousarray(to_layout(V))).cuda())
                torch.cuda.synchronize()
            assert rel(U.cpu().numpy(), to_layout(oracle.r2c3d(u))) < tol, (nx, ny, nz)
            assert rel(b.cpu().numpy(), oracle.c2r3d(V, nx)) < tol, (nx, ny, nz)
