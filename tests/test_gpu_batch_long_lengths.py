"""Batches with lengths above 324: fused launches over classes of long lengths (336 ..
512, 525 .. 720, 729 .. 1024) where a length has few workgroups, a launch of its own
from 1024 on.  Every length of the table in X, Y and Z, both precisions and layouts:
the fused launches equal the serial chains bit for bit and match the FP64 oracle.

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

LENGTHS = [n for n in synth.smooth7(325, 1024) if n not in (343, 686)]
DIMS = ([(n, 6, 3) for n in LENGTHS] + [(8, n, 3) for n in LENGTHS] + [(6, 5, n) for n in LENGTHS] +
        [(320, 64, 336), (300, 60, 336),    # 1300 tiles of length 336 along Z: a launch of its own
         (48, 343, 5), (686, 3, 10)])       # runtime-radix


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("stride1", [1, 0])
@pytest.mark.parametrize("prec", [pf.PF_F32, pf.PF_F64], ids=["f32", "f64"])
def test_fused_matches_serial_and_oracle(prec, stride1):
    assert len(LENGTHS) == 56
    f64 = prec == pf.PF_F64
    tol = 1e-14 if f64 else 1e-6
    to_layout = oracle.to_stride1 if stride1 else (lambda a: a)
    print(f"case batch long lengths f64={f64} stride1={stride1}", flush=True)
    with pf.Batch(DIMS, pf.Layout(precision=prec, stride1=stride1), mode=pf.PF_BATCH_FUSED) as b:
        R, C, back = b.empty(0).zero_(), b.empty(1).zero_(), b.empty(0).zero_()
        for i, (nx, ny, nz) in enumerate(DIMS):
            b.view(R, 0, i).copy_(torch.from_numpy(synth.uniform(i, (nz, ny, nx)).astype(
                np.float64 if f64 else np.float32)))
        b.ftran(R, C)
        b.btran(C, back)
        b.set_mode(pf.PF_BATCH_SERIAL)
        C2, back2 = b.empty(1).zero_(), b.empty(0).zero_()
        b.ftran(R, C2)
        b.btran(C, back2)
        torch.cuda.synchronize()
        assert torch.equal(C2, C) and torch.equal(back2, back)
        for i, (nx, ny, nz) in enumerate(DIMS):
            u = b.view(R, 0, i).cpu().numpy()
            assert rel(b.view(C, 1, i).cpu().numpy(), to_layout(oracle.r2c3d(u))) < tol, DIMS[i]
            assert rel(b.view(back, 0, i).cpu().numpy() / u.size, u) < tol, DIMS[i]
