"""The workloads this library is timed on.

A case is one pass of a user's program over data it already holds on the GPU,
through the package's public entry points:

  pair      forward R2C, then backward C2R, of one grid with one plan: the work
            of a pseudo-spectral time step (and of the paper's own benchmark).
  inplace   the same on one in-place buffer; the program puts its field into
            the buffer first, as the transforms consume it.
  batch     forward and backward of many grids of different sizes at once.
  spectral  the differentiable Chebyshev spectral step with its gradient.

Grids are (nx, ny, nz), x fastest.  Sizes come from the repository's smoke
check, tests and benchmark; the drawn ones are any 7-smooth lengths of the same
range.  Fields are a few energetic large scales over a floor of small-scale
noise, as in a turbulence run.
"""
import math

import torch

import paper_1905_02803_amd as pf


def listed():
    return [
        # Smallest calls: launches and host time.  A unit-cell or test-sized box (the smoke check's grid).
        _pair("tiny_36x20x24_f32", 36, 20, 24),
        # A small box in double precision, the paper's own precision: many steps of a small direct simulation.
        _pair("small_64x64x64_f64", 64, 64, 64, "f64"),
        # An ordinary single-precision box that the last-level cache holds.
        _pair("mid_256x256x256_f32", 256, 256, 256),
        # An ordinary grid with unequal, non-power-of-two edges (a channel- or duct-like box).
        _pair("mixed_480x360x250_f32", 480, 360, 250),
        # The same kind of grid in double precision.
        _pair("mixed_300x280x250_f64", 300, 280, 250, "f64"),
        # Natural-order output ([nz][ny][nxh], STRIDE1 undefined) on a 3 * 2^k grid: programs that index modes as fields.
        _pair("natural_384x384x384_f32", 384, 384, 384, stride1=0),
        # Power-of-two boxes of isotropic-turbulence runs, both precisions.
        _pair("pow2_512x512x512_f32", 512, 512, 512),
        _pair("pow2_512x512x512_f64", 512, 512, 512, "f64"),
        # A large 3 * 2^k box, the usual step between two powers of two.
        _pair("large_768x768x384_f32", 768, 768, 384),
        # The headline grid.
        _pair("pow2_1024x1024x1024_f32", 1024, 1024, 1024),
        # Many independent grids of different sizes (ensembles, adaptive patches), the batch's default mode.
        dict(name="batch32_48to320_f32", kind="batch", count=32, lo=48, hi=320, pick=4, dtype="f32"),
        # Differentiable spectral step, wall-bounded in z (Chebyshev), forward and gradient: a training step's layer.
        dict(name="spectral_512x512x257_f32", kind="spectral", nx=512, ny=512, nz=257, dtype="f32"),
    ]


def _pair(name, nx, ny, nz, dtype="f32", stride1=1, third="fft", inplace=0):
    return dict(name=name, kind="pair", nx=nx, ny=ny, nz=nz, dtype=dtype, stride1=stride1, third=third,
                inplace=inplace)


def _smooth7(lo, hi):
    out = []
    for n in range(lo, hi + 1):
        m = n
        for p in (2, 3, 5, 7):
            while m % p == 0:
                m //= p
        if m == 1:
            out.append(n)
    return out


def _near(rng, x, lo, hi):
    """A 7-smooth length near x (any of the six nearest, so odd ones come up)."""
    s = sorted(_smooth7(lo, hi), key=lambda n: abs(math.log(n / x)))
    return rng.choice(s[:6])


def _edges(rng, lo, hi, count, most):
    """`count` edges around one size spread over its logarithm, within a factor of two of it, most points in all."""
    while True:
        base = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        e = [_near(rng, min(hi, max(lo, base * 2.0 ** rng.uniform(-1, 1))), lo, hi) for _ in range(count)]
        if math.prod(e) <= most:
            return e


def draw(rng):
    dtype = rng.choice(["f32", "f32", "f64"])
    most = (1 << 28) if dtype == "f32" else (1 << 26)
    what = rng.random()
    if what < 0.68:
        nx, ny, nz = _edges(rng, 20, 1024, 3, most)
        c = _pair("", nx, ny, nz, dtype, stride1=rng.choice([1, 1, 1, 0]),
                  third=rng.choice(["fft"] * 5 + ["empty"]), inplace=rng.choice([0, 0, 0, 1]))
    elif what < 0.84:
        lo = rng.choice([24, 48, 48])
        c = dict(kind="batch", count=rng.randint(4, 32), lo=lo, hi=rng.randint(2 * lo, 320 if dtype == "f32" else 200),
                 pick=rng.randint(0, 1 << 20), dtype=dtype)
    else:
        nx, ny, m = _edges(rng, 24, 512, 3, most // 2)
        c = dict(kind="spectral", nx=nx, ny=ny, nz=m + 1, dtype=dtype)
    c.pop("name", None)
    return c


# ---- a user's program -------------------------------------------------------

_REAL = {"f32": torch.float32, "f64": torch.float64}
_THIRD = {"fft": pf.PF_THIRD_FFT, "empty": pf.PF_THIRD_EMPTY}


def _layout(case):
    return dict(precision=pf.PF_F64 if case["dtype"] == "f64" else pf.PF_F32)


def _field(gen, nx, ny, nz, dtype):
    """Large scales (random phases and wavevectors up to 3 per edge) plus noise, [nz][ny][nx]."""
    u = torch.randn((nz, ny, nx), generator=gen, device="cuda", dtype=dtype).mul_(0.2)
    x, y, z = (torch.arange(n, device="cuda", dtype=dtype) * (2 * math.pi / n) for n in (nx, ny, nz))
    k = torch.randint(0, 4, (4, 3), generator=gen, device="cuda").to(dtype)
    ph = torch.rand((4, 3), generator=gen, device="cuda", dtype=dtype) * (2 * math.pi)
    for i in range(4):
        plane = torch.cos(k[i, 1] * y + ph[i, 1])[:, None] * torch.cos(k[i, 0] * x + ph[i, 0])
        u.addcmul_(torch.cos(k[i, 2] * z + ph[i, 2])[:, None, None], plane)
    return u


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _batch_dims(case):
    """The batch's grids, from the case alone (a small multiplicative generator: no library's stream)."""
    s, x, out = _smooth7(case["lo"], case["hi"]), case["pick"] * 2 + 1, []
    for _ in range(case["count"]):
        e = []
        for _ in range(3):
            x = (x * 6364136223846793005 + 1442695040888963407) % (1 << 64)
            e.append(s[(x >> 33) % len(s)])
        out.append(tuple(e))
    return out


def prepare(case, seed):
    gen, dtype = _generator(seed), _REAL[case["dtype"]]
    if case["kind"] == "batch":
        dims = _batch_dims(case)
        batch = pf.Batch(dims, pf.Layout(**_layout(case)))
        real, spec, back = (batch.empty(which) for which in (0, 1, 0))
        for i, (nx, ny, nz) in enumerate(dims):
            batch.view(real, 0, i).copy_(_field(gen, nx, ny, nz, dtype))
        return dict(case=case, batch=batch, real=real, spec=spec, back=back)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    u = _field(gen, nx, ny, nz, dtype)
    if case["kind"] == "spectral":
        plan = pf.Plan(nx, ny, nz, third=pf.PF_THIRD_CHEB, **_layout(case))
        g = torch.randn((nz, ny, nx), generator=gen, device="cuda", dtype=dtype)
        return dict(case=case, plan=plan, u=u.requires_grad_(), g=g)
    plan = pf.Plan(nx, ny, nz, stride1=case["stride1"], third=_THIRD[case["third"]], inplace=case["inplace"],
                   **_layout(case))
    if case["inplace"]:
        buf = torch.empty(plan.inplace_bytes // u.element_size(), dtype=dtype, device="cuda")
        return dict(case=case, plan=plan, u=u, buf=buf)
    return dict(case=case, plan=plan, u=u, U=plan.empty_complex(), r=plan.empty_real())


def run(state):
    kind = state["case"]["kind"]
    if kind == "batch":
        b = state["batch"]
        b.ftran(state["real"], state["spec"])
        b.btran(state["spec"], state["back"])
        n = len(b.dims)
        return [b.view(state["spec"], 1, i) for i in range(n)], [b.view(state["back"], 0, i) for i in range(n)]
    plan, u = state["plan"], state["u"]
    if kind == "spectral":
        y = pf.spectral_step_autograd(u, plan)
        (du,) = torch.autograd.grad(y, u, state["g"])
        return y.detach(), du
    if state["case"]["inplace"]:
        buf = state["buf"]
        field = buf[:u.numel()].view(u.shape)
        field.copy_(u)
        plan.ftran_inplace(buf)
        plan.btran_inplace(buf)
        return field
    plan.ftran(u, state["U"])
    plan.btran(state["U"], state["r"])
    return state["U"], state["r"]


def work(case):
    """One pass: each input read once, each output written once; 2.5 N log2 N operations per real transform."""
    s = 8 if case["dtype"] == "f64" else 4

    def pair(nx, ny, nz, zlen):
        n, m = nx * ny * nz, (nx // 2 + 1) * ny * nz
        return 2 * (n * s + m * 2 * s), 2 * 2.5 * n * math.log2(max(2, nx * ny * zlen))

    if case["kind"] == "batch":
        each = [pair(nx, ny, nz, nz) for nx, ny, nz in _batch_dims(case)]
        return {"bytes": sum(e[0] for e in each), "flops": sum(e[1] for e in each)}
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if case["kind"] == "spectral":  # u -> y and g -> du; each is a forward and a backward transform
        return {"bytes": 4 * nx * ny * nz * s, "flops": 2 * pair(nx, ny, nz, 2 * (nz - 1))[1]}
    b, f = pair(nx, ny, nz, nz if case["third"] == "fft" else 1)
    if case["inplace"]:  # field -> buffer -> field, the spectrum an intermediate
        b = 2 * nx * ny * nz * s
    return {"bytes": b, "flops": f}


# ---- the same in 64 bits, without the library --------------------------------

def _exact_pair(u, stride1, third):
    u = u.double()
    axes = (0, 1, 2) if third == "fft" else (1, 2)
    U = torch.fft.rfftn(u, dim=axes)
    scale = math.prod(u.shape[a] for a in axes)
    if stride1:
        U = U.permute(2, 1, 0).contiguous()
    return U, u * scale


def _dct1(x):
    """Type-I DCT along the first axis: Y[k] = x[0] + (-1)^k x[n-1] + 2 sum x[j] cos(pi j k / (n-1))."""
    n = x.shape[0]
    return torch.fft.fft(torch.cat([x, x[1:n - 1].flip(0)]), dim=0)[:n]


def _spectral(v, adjoint):
    """s B(m F v) (its transpose when adjoint): the x derivative of the inverse Laplacian, Chebyshev along z."""
    nz, ny, nx = v.shape
    w = torch.full((nz, 1, 1), 2.0, dtype=torch.float64, device=v.device)
    w[0] = w[-1] = 1.0
    v = v.double() / w if adjoint else v.double()
    kx = torch.arange(nx // 2 + 1, device=v.device, dtype=torch.float64) * (2 * math.pi / nx)
    ky = torch.arange(ny, device=v.device, dtype=torch.float64)
    ky = torch.where(2 * ky <= ny, ky, ky - ny) * (2 * math.pi / ny)
    kz = torch.arange(nz, device=v.device, dtype=torch.float64) * (math.pi / (nz - 1))
    k2 = kx ** 2 + ky[:, None] ** 2 + kz[:, None, None] ** 2
    mu = torch.where(k2 > 0, -kx / k2, torch.zeros_like(k2))
    m = torch.complex(torch.zeros_like(mu), -mu if adjoint else mu)
    U = _dct1(torch.fft.rfftn(v, dim=(1, 2))) * m
    U = torch.fft.ifft(_dct1(U), dim=1, norm="forward")
    U[..., 0].imag.zero_()  # the last step uses the real parts of modes 0 and nx / 2
    if nx % 2 == 0:
        U[..., -1].imag.zero_()
    out = torch.fft.irfft(U, n=nx, dim=2, norm="forward") / (nx * ny * 2 * (nz - 1))
    return out * w if adjoint else out


def exact(case, seed):
    gen, dtype = _generator(seed), _REAL[case["dtype"]]
    if case["kind"] == "batch":
        both = [_exact_pair(_field(gen, nx, ny, nz, dtype), 1, "fft") for nx, ny, nz in _batch_dims(case)]
        return [b[0] for b in both], [b[1] for b in both]
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    u = _field(gen, nx, ny, nz, dtype)
    if case["kind"] == "spectral":
        g = torch.randn((nz, ny, nx), generator=gen, device="cuda", dtype=dtype)
        return _spectral(u, False), _spectral(g, True)
    U, r = _exact_pair(u, case["stride1"], case["third"])
    return r if case["inplace"] else (U, r)
