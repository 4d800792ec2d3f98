"""Mixed-radix passes on workspaces above and below 128 MB, where the backward Z
pass changes the order of its workgroups (ky first above) and the passes that
write the user arrays take non-temporal stores (up to 320 MB), both layouts and
precisions, ragged last column blocks included, against the FP64 oracle.

Bounds on the relative L2 error: 1e-6 in FP32, 1e-14 in FP64 (at most 10
butterfly levels per axis over 3 axes, each contributing below 1.5 ulp).
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1905_02803_amd as pf  # noqa: E402


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("stride1", [1, 0])
@pytest.mark.parametrize("nx,ny,nz,f64", [
    (300, 288, 320, False),  # 112 MB
    (300, 350, 320, False),  # 137 MB
    (300, 486, 480, False),  # 285 MB
    (300, 486, 560, False),  # 332 MB
    (600, 288, 512, False),  # 342 MB: backward Z of length 512 on this kernel
    (600, 144, 512, True),   # 342 MB, likewise
    (200, 250, 300, True),   # 119 MB
    (210, 250, 324, True),   # 138 MB
    (150, 480, 486, True),   # 285 MB
])
def test_against_oracle(nx, ny, nz, f64, stride1):
    tol = 1e-14 if f64 else 1e-6
    print(f"case workspace order {nx}x{ny}x{nz} f64={f64} stride1={stride1}", flush=True)
    u = synth.uniform(nx + stride1, (nz, ny, nx)).astype(np.float64 if f64 else np.float32)
    V = synth.complex_half(ny + stride1, (nz, ny, nx // 2 + 1)).astype(np.complex128 if f64 else np.complex64)
    to_layout = oracle.to_stride1 if stride1 else (lambda a: a)
    with pf.Plan(nx, ny, nz, pf.Layout(stride1=stride1, precision=pf.PF_F64 if f64 else pf.PF_F32)) as plan:
        if nz == 512:
            assert plan.pass_kernel(pf.PF_DIR_BACKWARD, 0) == ("c2c_mixed" if stride1 else "c2c_pow2")
            assert plan.pass_kernel(pf.PF_DIR_FORWARD, 2) == "c2c_pow2"
        U = plan.ftran(torch.from_numpy(u).cuda())
        b = plan.btran(torch.from_numpy(np.ascontiguousarray(to_layout(V))).cuda())
        torch.cuda.synchronize()
    assert rel(U.cpu().numpy(), to_layout(oracle.r2c3d(u))) < tol
    assert rel(b.cpu().numpy(), oracle.c2r3d(V, nx)) < tol
