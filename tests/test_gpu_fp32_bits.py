"""FP32 forward results of the mixed-radix passes, bit for bit.

On a large grid with a few energetic modes over noise the rounding of the
energetic lines shows in the weak modes (1e-3 of the noise at 768 x 768 x 384),
so another order of the same sums moves them visibly.  The rounding is therefore
fixed:

* lengths on a staged plan (17 .. 45, above 320 but 360 and 480) round as the
  runtime-radix kernels do, which a batch with narrow tiles runs;
* the others (48 .. 320, 360, 480) give the CRC-32 in golden/fp32_forward_crc.txt
  (per length the X, Y and Z pass on uniform fields), taken from the kernels
  that first ran them.

The energetic field is also held to the per-shell bounds against the FP64 oracle.
"""
import os
import zlib

import numpy as np
import pytest

import oracle
import synth
from tests import errbounds

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1905_02803_amd as pf  # noqa: E402

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "fp32_forward_crc.txt")
STAGED = [n for n in synth.smooth7(17, 1024) if (n < 48 or n > 320) and n not in (343, 360, 480, 686)]


def roles(n):
    """(nx, ny, nz) with length n in X, Y, Z and lengths below 16 (runtime-radix) elsewhere."""
    return (n, 6, 4), (8, n, 4), (8, 4, n)


def field(n, nx, ny, nz):
    return torch.from_numpy(synth.uniform(500 + n, (nz, ny, nx)).astype(np.float32)).cuda()


def runtime_radix(u, nx, ny, nz):
    """Forward by the runtime-radix kernels: a batch of one with 8-column tiles."""
    with pf.Batch([(nx, ny, nz)], pf.Layout(), tune=[((0, 0, 0), (8, 8, 8))]) as b:
        R, C = b.empty(0), b.empty(1)
        b.view(R, 0, 0).copy_(u)
        b.ftran(R, C)
        return b.view(C, 1, 0).clone()


@pytest.mark.parametrize("part", range(4))
def test_staged_lengths_round_as_the_runtime_radix_kernels(part):
    for n in STAGED[part::4]:
        for nx, ny, nz in roles(n):
            if nx in (512, 1024) or ny in (512, 1024) or nz in (512, 1024):
                continue  # a plan runs these on the power-of-two kernels
            print(f"case fp32 bits {nx}x{ny}x{nz}", flush=True)
            u = field(n, nx, ny, nz)
            with pf.Plan(nx, ny, nz) as plan:
                assert torch.equal(plan.ftran(u), runtime_radix(u, nx, ny, nz)), (nx, ny, nz)


def test_two_step_lengths_give_the_golden_bits():
    with open(GOLDEN) as f:
        golden = [line.split() for line in f if line.strip() and not line.startswith("#")]
    assert len(golden) == 58
    for n, *want in golden:
        n = int(n)
        for (nx, ny, nz), crc in zip(roles(n), want):
            print(f"case fp32 bits {nx}x{ny}x{nz}", flush=True)
            with pf.Plan(nx, ny, nz) as plan:
                U = plan.ftran(field(n, nx, ny, nz)).cpu().numpy()
            assert f"{zlib.crc32(U.tobytes()):08x}" == crc, (nx, ny, nz)


@pytest.mark.timeout(600)
def test_energetic_modes_over_noise():
    """Four modes of amplitude 1 over noise of 0.2 at 768 x 768 x 384."""
    nx, ny, nz = 768, 768, 384
    print(f"case fp32 energetic modes {nx}x{ny}x{nz}", flush=True)
    rng = np.random.default_rng(11)
    u = synth.uniform(12, (nz, ny, nx)).astype(np.float32) * np.float32(0.2)
    x, y, z = (2 * np.pi * np.arange(n) / n for n in (nx, ny, nz))
    for k in rng.integers(0, 4, (4, 3)):
        a, b, c = rng.uniform(0, 2 * np.pi, 3)
        plane = np.cos(k[1] * y + b)[:, None] * np.cos(k[0] * x + a)
        u += (np.cos(k[2] * z + c)[:, None, None] * plane).astype(np.float32)
    ud = torch.from_numpy(u).cuda()
    with pf.Plan(nx, ny, nz) as plan:
        U = plan.ftran(ud)
    assert torch.equal(U, runtime_radix(ud, nx, ny, nz))
    for lo, hi, m, e, bound in errbounds.check_shells(U.cpu().numpy(), oracle.to_stride1(oracle.r2c3d(u)), nx, ny, nz,
                                                      1e-6):
        print(f"  shell [{lo:g}, {hi:g}): {m} modes, rel L2 {e:.3e} (bound {bound:.3e})", flush=True)
