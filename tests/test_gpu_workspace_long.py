"""Long mixed-radix lengths, whose tiles go through LDS in halves (above 80 KB) and
whose FP64 X tiles hold two line pairs, on workspaces large enough for what
depends on the size: above 64 MB X and Y passes without runs of tiles per XCD, from
128 to 320 MB non-temporal stores of the user's arrays and (STRIDE1, above 128 MB)
ky-first order of the backward Z pass.  Both layouts, against the FP64 oracle.

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
    (100, 360, 768, False),   # Z of three steps, 141 MB
    (100, 300, 864, False),   # Z of two steps in halves, 133 MB
    (100, 324, 1008, False),  # 167 MB
    (60, 300, 1000, True),    # 154 MB
    (60, 324, 980, True),     # 163 MB
    (90, 768, 300, False),    # Y of three steps, 88 MB
    (90, 900, 300, False),    # Y of two steps in halves, 104 MB
    (60, 1000, 150, True),    # 77 MB
    (1008, 200, 180, False),  # X of three steps, 147 MB
    (972, 210, 162, False),   # X of two steps, 135 MB
    (1000, 112, 150, True),   # X with two line pairs per tile, 135 MB
    (735, 147, 175, True),    # an odd one, 152 MB
])
def test_against_oracle(nx, ny, nz, f64, stride1):
    tol = 1e-14 if f64 else 1e-6
    print(f"case workspace long {nx}x{ny}x{nz} f64={f64} stride1={stride1}", flush=True)
    u = synth.uniform(nx + stride1, (nz, ny, nx)).astype(np.float64 if f64 else np.float32)
    V = synth.complex_half(ny + stride1, (nz, ny, nx // 2 + 1)).astype(np.complex128 if f64 else np.complex64)
    to_layout = oracle.to_stride1 if stride1 else (lambda a: a)
    with pf.Plan(nx, ny, nz, pf.Layout(stride1=stride1, precision=pf.PF_F64 if f64 else pf.PF_F32)) as plan:
        for d in (pf.PF_DIR_FORWARD, pf.PF_DIR_BACKWARD):
            assert {plan.pass_symbol(d, i) for i in range(3)} == {"k_mr_c2c", "k_mr_x"}
        U = plan.ftran(torch.from_numpy(u).cuda())
        b = plan.btran(torch.from_numpy(np.ascontiguousarray(to_layout(V))).cuda())
        torch.cuda.synchronize()
    assert rel(U.cpu().numpy(), to_layout(oracle.r2c3d(u))) < tol
    assert rel(b.cpu().numpy(), oracle.c2r3d(V, nx)) < tol
