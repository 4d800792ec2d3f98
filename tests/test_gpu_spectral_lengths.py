"""Spectral step on the compile-time mixed-radix z pass (extension lengths 2 (nz -
1) of 16 .. 1024 in the table; FP32 powers of two from 256 on have their own).

Step and adjoint against the FP64 oracle's composition with the multiplier
applied in numpy: the smallest and largest extension, lengths whose exchange
goes through LDS in halves (above 80 KB: 2 (nz - 1) = 768, 1000), odd nx and ny,
a ragged last column block, both Z-pencil layouts (the step never writes one).
Bounds on the relative L2 error: 1e-6 in FP32; in FP64 2e-14: six transform
axes of at most 10 butterfly levels, below 1.5 ulp (2.2e-16) each.
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


def multiplier(nx, ny, nz):
    kx = 2 * np.pi * np.arange(nx // 2 + 1) / nx
    k = np.arange(ny)
    ky = 2 * np.pi * np.where(2 * k <= ny, k, k - ny) / ny
    kz = np.pi * np.arange(nz) / (nz - 1)
    k2 = kx[None, None, :] ** 2 + ky[None, :, None] ** 2 + kz[:, None, None] ** 2
    with np.errstate(divide="ignore", invalid="ignore"):
        m = np.where(k2 > 0, -kx[None, None, :] / k2, 0.0)
    return 1j * m / (nx * ny * 2 * (nz - 1))


@pytest.mark.parametrize("prec", [pf.PF_F32, pf.PF_F64], ids=["f32", "f64"])
@pytest.mark.parametrize("ext", [16, 18, 36, 50, 64, 98, 128, 250, 294, 512, 768, 882, 1000, 1024])
def test_spectral_step_on_mixed_lengths(ext, prec):
    f64 = prec == pf.PF_F64
    nx, ny, nz, tol = 35, 6, ext // 2 + 1, 2e-14 if f64 else 1e-6
    print(f"case spectral {nx}x{ny}x{nz} f64={f64}", flush=True)
    dt = np.float64 if f64 else np.float32
    u = synth.uniform(ext, (nz, ny, nx)).astype(dt)
    M = multiplier(nx, ny, nz)
    w = np.full((nz, 1, 1), 2.0)
    w[0] = w[-1] = 1.0
    with pf.Plan(nx, ny, nz, pf.Layout(precision=prec, third=pf.PF_THIRD_CHEB, stride1=(ext // 2) % 2)) as plan:
        ud = torch.from_numpy(u).cuda()
        step = pf.spectral_step(plan, ud).cpu().numpy()
        adj = pf.spectral_step(plan, ud, adjoint=True).cpu().numpy()
        assert np.array_equal(ud.cpu().numpy(), u)  # the input is left as it was
    assert rel(step, oracle.c2r3d_cheb(oracle.r2c3d_cheb(u) * M, nx)) < tol
    assert rel(adj, w * oracle.c2r3d_cheb(oracle.r2c3d_cheb(u / w) * np.conj(M), nx)) < tol
