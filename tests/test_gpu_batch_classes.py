"""Batched launches over classes of lengths (16 .. 112, 120 .. 243, 245 .. 324).

One batch holds the first and last length of every class in each role (X, Y,
Z), lengths whose step 1 takes two rounds (125, 175, 243, 245, 250), a length
above the classes (336, a launch of its own) and one below the table (10, the
runtime-radix kernels); the fused launches are compared with the FP64 oracle and,
bit for bit, with the serial chains (per-length kernels, the same arithmetic).
Bounds: 1e-6 in FP32; 1e-14 in FP64 (10 butterfly levels per axis, 3 axes, below
1.5 ulp each).
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1905_02803_amd as pf  # noqa: E402

DIMS = [(16, 112, 21), (112, 16, 120), (120, 10, 112), (243, 20, 18), (18, 243, 10), (24, 18, 243), (245, 16, 20),
        (20, 245, 16), (16, 21, 324), (324, 18, 16), (125, 18, 245), (18, 175, 125), (250, 125, 6), (336, 16, 18),
        (16, 18, 336), (10, 10, 10), (49, 50, 27)]


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("stride1", [1, 0])
@pytest.mark.parametrize("prec", [pf.PF_F32, pf.PF_F64], ids=["f32", "f64"])
def test_classes_match_oracle_and_serial(prec, stride1):
    f64 = prec == pf.PF_F64
    tol = 1e-14 if f64 else 1e-6
    to_layout = oracle.to_stride1 if stride1 else (lambda a: a)
    with pf.Batch(DIMS, pf.Layout(precision=prec, stride1=stride1), mode=pf.PF_BATCH_FUSED) as b:
        R, C = b.empty(0).zero_(), b.empty(1).zero_()
        for i, (nx, ny, nz) in enumerate(DIMS):
            b.view(R, 0, i).copy_(torch.from_numpy(synth.uniform(40 + i, (nz, ny, nx)).astype(
                np.float64 if f64 else np.float32)))
        print(f"case batch classes f64={f64} stride1={stride1}", flush=True)
        b.ftran(R, C)
        back = b.empty(0).zero_()
        b.btran(C, back)
        torch.cuda.synchronize()
        for i, (nx, ny, nz) in enumerate(DIMS):
            u = b.view(R, 0, i).cpu().numpy()
            ref = oracle.r2c3d(u)
            assert rel(b.view(C, 1, i).cpu().numpy(), to_layout(ref)) < tol, DIMS[i]
            assert rel(b.view(back, 0, i).cpu().numpy() / u.size, u) < tol, DIMS[i]
        b.set_mode(pf.PF_BATCH_SERIAL)
        C2, back2 = b.empty(1).zero_(), b.empty(0).zero_()
        b.ftran(R, C2)
        b.btran(C, back2)
        torch.cuda.synchronize()
        assert torch.equal(C2, C) and torch.equal(back2, back)
