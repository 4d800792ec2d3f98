"""C2C passes of length 256, which take the mixed-radix kernel before the
power-of-two one (FP64 with a power-of-two X pass keeps the latter): on the
transposed workspace, on blocks and ragged natural-order rows, against the FP64
oracle.

Bounds on the relative L2 error: 1e-6 in FP32, 1e-14 in FP64 (at most 11
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


@pytest.mark.parametrize("f64", [False, True], ids=["f32", "f64"])
@pytest.mark.parametrize("nx,ny,nz,stride1", [(512, 256, 20, 1), (512, 16, 256, 1), (512, 256, 256, 1),
                                              (1024, 48, 256, 1), (45, 256, 256, 1), (45, 256, 256, 0)])
def test_against_oracle(nx, ny, nz, stride1, f64):
    tol = 1e-14 if f64 else 1e-6
    print(f"case length 256 {nx}x{ny}x{nz} f64={f64} stride1={stride1}", flush=True)
    u = synth.uniform(nx + ny, (nz, ny, nx)).astype(np.float64 if f64 else np.float32)
    V = synth.complex_half(nx + nz, (nz, ny, nx // 2 + 1)).astype(np.complex128 if f64 else np.complex64)
    to_layout = oracle.to_stride1 if stride1 else (lambda a: a)
    with pf.Plan(nx, ny, nz, pf.Layout(stride1=stride1, precision=pf.PF_F64 if f64 else pf.PF_F32)) as plan:
        transposed = nx >= 512
        for d, i in ((pf.PF_DIR_FORWARD, 1), (pf.PF_DIR_FORWARD, 2), (pf.PF_DIR_BACKWARD, 0), (pf.PF_DIR_BACKWARD, 1)):
            if (nz if "_z_" in plan.pass_name(d, i) else ny) == 256:
                assert plan.pass_kernel(d, i) == ("c2c_pow2" if f64 and transposed else "c2c_mixed"), (d, i)
        U = plan.ftran(torch.from_numpy(u).cuda())
        b = plan.btran(torch.from_numpy(np.ascontiguousarray(to_layout(V))).cuda())
        torch.cuda.synchronize()
    assert rel(U.cpu().numpy(), to_layout(oracle.r2c3d(u))) < tol
    assert rel(b.cpu().numpy(), oracle.c2r3d(V, nx)) < tol


@pytest.mark.parametrize("f64", [False, True], ids=["f32", "f64"])
@pytest.mark.parametrize("nx,ny,nz", [(512, 256, 16), (512, 32, 256), (640, 256, 20), (600, 288, 512), (512, 320, 512)])
def test_processor_grid_blocks_are_the_same_bits(nx, ny, nz, f64):
    """The kernels of the m1 x m2 block layout, which never has the transposed
    workspace, are those of the 1 x 1 plan."""
    print(f"case length 256 blocks {nx}x{ny}x{nz} f64={f64}", flush=True)
    cdt, rdt, prec = (np.complex128, np.float64, pf.PF_F64) if f64 else (np.complex64, np.float32, pf.PF_F32)
    from tests.test_gpu_grid import blocks, unblocks

    nxh = nx // 2 + 1
    u = synth.uniform(nx + 7, (nz, ny, nx)).astype(rdt)
    with pf.Plan(nx, ny, nz, pf.Layout(precision=prec)) as full:
        U = full.ftran(torch.from_numpy(u).cuda())
        b = full.btran(U).cpu().numpy()  # [z][y][x]
        U = U.cpu().numpy()  # [kx][ky][kz]
    lay = pf.Layout(m1=2, m2=3, precision=prec)
    with pf.Plan(nx, ny, nz, lay) as grid:
        ub = torch.from_numpy(blocks(u.transpose(2, 1, 0), nx, ny, nz, lay, pf.PF_PENCIL_X)).cuda()
        out = torch.empty(nxh * ny * nz, dtype=getattr(torch, np.dtype(cdt).name), device="cuda")
        back = torch.empty_like(ub)
        pf.pf_ftran_r2c(grid.handle, ub.data_ptr(), out.data_ptr(), 0)
        pf.pf_btran_c2r(grid.handle, out.data_ptr(), back.data_ptr(), 0)
        torch.cuda.synchronize()
    assert np.array_equal(unblocks(out.cpu().numpy(), (nxh, ny, nz), nx, ny, nz, lay, pf.PF_PENCIL_Z), U)
    got = unblocks(back.cpu().numpy(), (nx, ny, nz), nx, ny, nz, lay, pf.PF_PENCIL_X)
    assert np.array_equal(got, b.transpose(2, 1, 0))
