"""Timed workloads of the pseudospectral solver, through its public Plan calls.

A case is one call of a user's program on resident device data:
  step       rk2_step (NS or MHD, one box or a grid nx x ny x nz), `steps` steps per call
  ensemble   rk2_step of many uneven boxes in one plan
  nonlinear  nonlinear_ns / nonlinear_mhd (a user's own integrator)
  r2c, c2r   the batched 3D transforms of all fields, each direction
  spectrum   energy_spectrum of all fields, or the MHD diagnostics (mhd_spectrum)

`mode` says how the program set its plan up: "plain" keeps every default (any
input is valid, no plan-time search), "tuned" does what the benchmark does for a
dealiased solenoidal state: dealias pruning, the divergence form (FP64 NS keeps
the rotational one) and the autotuner.

Inputs: solenoidal random fields with a k^(-5/3) tail that fill the 2/3 sphere,
total energy 0.5 per field set; time step and viscosity follow the resolution
(dt = 0.2 / n, nu = 0.5 / n), so a state can be stepped for as long as one likes.
"""
import math

import torch

from paper_1003_4322_amd import binding

SIZES = (8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024)
ENSEMBLE = "64*48,96*16,128*4"


def _case(name, op, model, dims, dtype, mode="plain", steps=1, rot=False):
    nx, ny, nz = dims
    return {"name": name, "op": op, "model": model, "nx": nx, "ny": ny, "nz": nz, "dtype": dtype,
            "mode": mode, "steps": steps, "rot": rot, "boxes": ""}


def listed():
    cube = lambda n: (n, n, n)  # noqa: E731
    ens = _case("ensemble_ns_f32", "ensemble", "ns", cube(128), "f32", "tuned")
    ens["boxes"] = ENSEMBLE
    return [
        # the smallest problem of the repository: one step per call, where launches and latency count
        _case("step_ns32_f64", "step", "ns", cube(32), "f64"),
        # a small MHD run, ten steps between outputs
        _case("step_mhd64_f32", "step", "mhd", cube(64), "f32", "tuned", steps=10),
        # 48 x 64^3 + 16 x 96^3 + 4 x 128^3 independent boxes, one step of all of them
        ens,
        # a first run on a plan as it comes, in double precision, radix-3 size
        _case("step_ns192_f64", "step", "ns", cube(192), "f64"),
        # the 256^3 run with an output every ten steps
        _case("step_ns256_f32", "step", "ns", cube(256), "f32", "tuned", steps=10),
        # a box of unequal axes in a rotating frame
        _case("step_mhd_grid_f32", "step", "mhd", (256, 192, 384), "f32", "tuned", rot=True),
        # the 512^3 MHD run of the benchmark
        _case("step_mhd512_f32", "step", "mhd", cube(512), "f32", "tuned"),
        # the largest box: 1024^3
        _case("step_ns1024_f32", "step", "ns", cube(1024), "f32", "tuned"),
        # the nonlinear term alone, for a caller's own time integrator
        _case("nonlinear_mhd128_f64", "nonlinear", "mhd", cube(128), "f64"),
        # a physical field into the solver
        _case("r2c_ns384_f32", "r2c", "ns", cube(384), "f32"),
        # a state back into physical space
        _case("c2r_ns96_f64", "c2r", "ns", cube(96), "f64"),
        # diagnostics of an MHD run between steps
        _case("spectrum_mhd512_f32", "spectrum", "mhd", cube(512), "f32"),
    ]


def _mhd_ok(nx, dtype):
    return nx <= (1024 if dtype == "f32" else 512)


def draw(rng):
    """One more case: any operation, cubes and grids of 16^3 to about 400^3 points."""
    op = rng.choice(["step"] * 6 + ["ensemble", "nonlinear", "nonlinear", "r2c", "c2r", "spectrum"])
    dtype = rng.choice(["f32", "f32", "f64"])
    model = rng.choice(["ns", "mhd"])
    mode = rng.choice(["plain", "tuned"]) if op in ("step", "ensemble", "nonlinear") else "plain"
    steps = rng.choice([1, 1, 2, 5]) if op in ("step", "ensemble") else 1
    if op == "ensemble":
        counts = {}
        for n in sorted(rng.sample([16, 24, 32, 48, 64, 96, 128], 3)):
            counts[n] = max(1, int(2 ** rng.uniform(0, 5) * min(1.0, (96 / n) ** 3)))
        c = _case("", op, "ns", (max(counts),) * 3, dtype, mode, steps)
        c["boxes"] = ",".join("%d*%d" % (n, k) for n, k in sorted(counts.items()))
    else:
        edge = 2 ** (rng.uniform(12, 26) / 3)
        if rng.random() < 0.5:
            n = min(SIZES, key=lambda s: abs(math.log(s / edge)))
            dims = [n, n, n]
        else:
            near = [s for s in SIZES if edge / 3 <= s <= edge * 3]
            dims = [rng.choice(near) for _ in range(3)]
            while dims[0] * dims[1] * dims[2] > 2 ** 26:  # the longest axis gives way
                i = dims.index(max(dims))
                dims[i] = max(s for s in SIZES if s < dims[i])
        if model == "mhd" and not _mhd_ok(dims[0], dtype):
            model = "ns"
        rot = op == "step" and rng.random() < 0.25
        if dims[0] * dims[1] * dims[2] > 2 ** 24:
            steps = 1
        c = _case("", op, model, dims, dtype, mode, steps, rot)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _boxes(case):
    """(nx, ny, nz) of every box."""
    if not case["boxes"]:
        return [(case["nx"], case["ny"], case["nz"])]
    out = []
    for part in case["boxes"].split(","):
        n, k = part.split("*")
        out += [(int(n),) * 3] * int(k)
    return out


def _lengths(case):
    """Box lengths over 2 pi: a rotating-frame case runs in a box twice as tall."""
    return (1.0, 1.0, 2.0) if case["rot"] else (1.0, 1.0, 1.0)


def _omega(case):
    return (0.0, 0.0, 2.0) if case["rot"] else (0.0, 0.0, 0.0)


def _params(case):
    n = max(max(d) for d in _boxes(case))
    nu = 0.5 / n
    return nu, 0.7 * nu if case["model"] == "mhd" else 0.0, 0.2 / n


def _index(n, half=False):
    """Signed wavenumber of every storage index of an axis."""
    k = torch.arange(n // 2 + 1 if half else n, device="cuda")
    return k if half else torch.where(k < n // 2, k, k - n)


def _kept(dims):
    """The 2/3 rule: (3 kx/nx)^2 + (3 ky/ny)^2 + (3 kz/nz)^2 < 1, in integers."""
    nx, ny, nz = dims
    m = math.lcm(nx, ny, nz)
    x, y, z = ((m // n) * _index(n, i == 0) for i, n in enumerate(dims))
    return 9 * (x[None, None, :] ** 2 + y[None, :, None] ** 2 + z[:, None, None] ** 2) < m * m


def _wavenumbers(dims, lengths, dtype):
    """Physical wavenumbers along x, y, z, shaped to broadcast over [kz][ky][kx]."""
    x, y, z = (_index(n, i == 0).to(dtype) / lengths[i] for i, n in enumerate(dims))
    return x[None, None, :], y[None, :, None], z[:, None, None]


def _solenoidal(dims, lengths, gen, dtype):
    """Random velocity-like half spectra [3][kz][ky][kx <= nx/2], energy 0.5."""
    nx, ny, nz = dims
    real = torch.float32 if dtype == torch.complex64 else torch.float64
    kx, ky, kz = _wavenumbers(dims, lengths, real)
    a = [torch.randn((nz, ny, nx // 2 + 1), dtype=dtype, device="cuda", generator=gen) for _ in range(3)]
    # E(k) ~ k^4 below k0, k^(-5/3) above it, zero outside the 2/3 sphere
    shape = (1 + (kx * kx + ky * ky + kz * kz) / 9.0) ** (-17.0 / 12.0) * _kept(dims)
    v = torch.empty((3, nz, ny, nx // 2 + 1), dtype=dtype, device="cuda")
    v[0] = (ky * a[2] - kz * a[1]) * shape
    v[1] = (kz * a[0] - kx * a[2]) * shape
    v[2] = (kx * a[1] - ky * a[0]) * shape
    del a, shape
    p = v[..., 0]  # a real field: v(-k) = conj v(k) on the kx = 0 plane
    v[..., 0] = 0.5 * (p + torch.roll(torch.flip(p, (1, 2)), (1, 1), (1, 2)).conj())
    energy = 0.0
    for f in v:
        energy += float(torch.view_as_real(f).square().sum()) - 0.5 * float(
            torch.view_as_real(f[..., 0]).square().sum())
    v *= math.sqrt(0.5 / energy)
    return v


def _state(case, seed):
    """The spectral state: u (NS) or z+ = u + b, z- = u - b (MHD); ensembles flat."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype = torch.complex64 if case["dtype"] == "f32" else torch.complex128
    sets = []
    for dims in _boxes(case):
        u = _solenoidal(dims, _lengths(case), gen, dtype)
        if case["model"] == "mhd":
            b = _solenoidal(dims, _lengths(case), gen, dtype)
            u = torch.cat((u + b, u - b))
        sets.append(u)
    return sets[0] if not case["boxes"] else torch.cat([s.reshape(-1) for s in sets])


def _real_fields(case, seed):
    """A physical field set [f][z][y][x]."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    real = torch.float32 if case["dtype"] == "f32" else torch.float64
    nf = 6 if case["model"] == "mhd" else 3
    return torch.randn((nf, case["nz"], case["ny"], case["nx"]), dtype=real, device="cuda", generator=gen)


def prepare(case, seed):
    mhd = case["model"] == "mhd"
    nf = 6 if mhd else 3
    model = binding.PS_MHD if mhd else binding.PS_NS
    x = _real_fields(case, seed) if case["op"] == "r2c" else _state(case, seed)
    dims = _boxes(case)
    if case["boxes"]:
        plan = binding.Plan([d[0] for d in dims], nf, case["dtype"])
    elif len(set(dims[0])) == 1:
        plan = binding.Plan(dims[0][0], nf, case["dtype"])
    else:
        plan = binding.Plan(nfields=nf, dtype=case["dtype"], grid=dims[0])
    if case["rot"]:
        plan.set_rotation(*_omega(case))
        plan.set_box(*(2 * math.pi * s for s in _lengths(case)))
    if case["mode"] == "tuned" and case["op"] in ("step", "ensemble", "nonlinear"):
        plan.set_variant("prune", 1)
        plan.set_variant("form", 0 if case["dtype"] == "f64" and not mhd else 1)
        plan.autotune(x, model, 3)
    return {"case": case, "plan": plan, "x": x, "model": model, "params": _params(case)}


def run(state):
    case, plan, x = state["case"], state["plan"], state["x"]
    op = case["op"]
    if op in ("step", "ensemble"):
        nu, eta, dt = state["params"]
        return plan.rk2_step(x, state["model"], nu, eta, dt, case["steps"])
    if op == "nonlinear":
        return plan.nonlinear_mhd(x) if case["model"] == "mhd" else plan.nonlinear_ns(x)
    if op == "r2c":
        return plan.fft_r2c(x)
    if op == "c2r":
        return plan.fft_c2r(x)
    return plan.mhd_spectrum(x) if case["model"] == "mhd" else plan.energy_spectrum(x)


def work(case):
    nf = 6 if case["model"] == "mhd" else 3
    c = 8 if case["dtype"] == "f32" else 16
    transforms = 14 if case["model"] == "mhd" else 8  # real 3D transforms per nonlinear term
    by = fl = 0.0
    for nx, ny, nz in _boxes(case):
        spectral = nf * nz * ny * (nx // 2 + 1) * c
        n3 = nx * ny * nz
        fft = 2.5 * n3 * math.log2(n3)
        if case["op"] in ("step", "ensemble"):
            by += 2 * spectral
            fl += 2 * case["steps"] * transforms * fft
        elif case["op"] == "nonlinear":
            by += 2 * spectral
            fl += transforms * fft
        elif case["op"] == "spectrum":
            by += spectral
            fl += 6 * spectral / c
        else:
            by += spectral + nf * n3 * c / 2
            fl += nf * fft
    return {"bytes": by, "flops": fl}


# ---------------------------------------------------------------------------
# The same results in 64 bits, from the equations
# ---------------------------------------------------------------------------
def _to_real(h, dims):
    nx, ny, nz = dims
    return torch.fft.irfftn(h, s=(nz, ny, nx), norm="forward")


def _cross(a, b):
    return [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]]


def _curl(h, k):
    return [1j * (k[1] * h[2] - k[2] * h[1]), 1j * (k[2] * h[0] - k[0] * h[2]),
            1j * (k[0] * h[1] - k[1] * h[0])]


def _project(n, k):
    k2 = k[0] * k[0] + k[1] * k[1] + k[2] * k[2]
    q = (k[0] * n[0] + k[1] * n[1] + k[2] * n[2]) / torch.where(k2 == 0, torch.ones_like(k2), k2)
    return [(n[i] - k[i] * q) * (k2 > 0) for i in range(3)]


def _nonlinear(z, mhd, dims, k, kept):
    """Rotational form: D P F[u x w (+ j x b)] (+- curl F[u x b] for MHD)."""
    fwd = lambda r: torch.fft.rfftn(r, norm="forward")  # noqa: E731
    uh = [0.5 * (z[i] + z[3 + i]) for i in range(3)] if mhd else [z[i] for i in range(3)]
    u = [_to_real(h, dims) for h in uh]
    w = [_to_real(h, dims) for h in _curl(uh, k)]
    p = _cross(u, w)
    del w
    if not mhd:
        return torch.stack([n * kept for n in _project([fwd(q) for q in p], k)])
    bh = [0.5 * (z[i] - z[3 + i]) for i in range(3)]
    b = [_to_real(h, dims) for h in bh]
    j = [_to_real(h, dims) for h in _curl(bh, k)]
    p = [x + y for x, y in zip(p, _cross(j, b))]
    del j
    n = _project([fwd(q) for q in p], k)
    del p
    e = _curl([fwd(q) for q in _cross(u, b)], k)
    return torch.stack([(n[i] + e[i]) * kept for i in range(3)] + [(n[i] - e[i]) * kept for i in range(3)])


def _rhs(z, mhd, dims, k, kept, nu, eta, omega):
    out = _nonlinear(z, mhd, dims, k, kept)
    k2 = k[0] * k[0] + k[1] * k[1] + k[2] * k[2]
    if any(omega):
        u = [0.5 * (z[i] + z[3 + i]) if mhd else z[i] for i in range(3)]
        w = _project([2 * c for c in _cross([float(o) for o in omega], u)], k)
        for f in range(out.shape[0]):
            out[f] -= w[f % 3]
    for f in range(out.shape[0]):
        if mhd:
            out[f] -= k2 * (0.5 * (nu + eta) * z[f] + 0.5 * (nu - eta) * z[(f + 3) % 6])
        else:
            out[f] -= nu * k2 * z[f]
    return out


def _shell_sums(values, dims):
    """values [kz][ky][kx] summed over the shells round(|k|) of the index, with the half-spectrum weights."""
    nx, ny, nz = dims
    x, y, z = (_index(n, i == 0) for i, n in enumerate(dims))
    k2 = x[None, None, :] ** 2 + y[None, :, None] ** 2 + z[:, None, None] ** 2
    s = torch.round(torch.sqrt(k2.double())).long()  # sqrt(integer) is never halfway between two integers
    top = round(math.sqrt((nx // 2) ** 2 + (ny // 2) ** 2 + (nz // 2) ** 2)) + 1
    w = torch.where((x == 0) | (2 * x == nx), 0.5, 1.0)[None, None, :]
    return torch.zeros(top, dtype=torch.float64, device="cuda").index_add_(0, s.reshape(-1), (values * w).reshape(-1))


def exact(case, seed):
    if any(nx * ny * nz > 512 ** 3 for nx, ny, nz in _boxes(case)):
        return None
    mhd = case["model"] == "mhd"
    op = case["op"]
    if op == "r2c":
        return torch.stack([torch.fft.rfftn(f.double()) for f in _real_fields(case, seed)])
    state = _state(case, seed)
    nu, eta, dt = _params(case)
    outs, at = [], 0
    for dims in _boxes(case):
        nx, ny, nz = dims
        nf = 6 if mhd else 3
        n = nf * nz * ny * (nx // 2 + 1)
        z = state.reshape(-1)[at:at + n].view(nf, nz, ny, nx // 2 + 1).to(torch.complex128)
        at += n
        k = _wavenumbers(dims, _lengths(case), torch.float64)
        if op == "c2r":
            return torch.stack([_to_real(f, dims) for f in z])
        if op == "spectrum":
            power = lambda fs: sum(f.real ** 2 + f.imag ** 2 for f in fs)  # noqa: E731
            if mhd:
                u, b = [0.5 * (z[i] + z[3 + i]) for i in range(3)], [0.5 * (z[i] - z[3 + i]) for i in range(3)]
                cross = sum(p.real * q.real + p.imag * q.imag for p, q in zip(u, b))
                spec = torch.stack([_shell_sums(v, dims) for v in (power(u), power(b), cross)])
                return spec, spec.sum(1)
            e = power(z)
            spec = _shell_sums(e, dims)
            z2 = _shell_sums(e * (k[0] ** 2 + k[1] ** 2 + k[2] ** 2), dims).sum()
            div = (k[0] * z[0] + k[1] * z[1] + k[2] * z[2]).abs().max()
            return spec, torch.stack([spec.sum(), z2, div])
        kept = _kept(dims)
        if op == "nonlinear":
            return _nonlinear(z, mhd, dims, k, kept)
        for _ in range(case["steps"]):
            mid = z + 0.5 * dt * _rhs(z, mhd, dims, k, kept, nu, eta, _omega(case))
            z = z + dt * _rhs(mid, mhd, dims, k, kept, nu, eta, _omega(case))
        outs.append(z)
    return outs[0] if not case["boxes"] else torch.cat([z.reshape(-1) for z in outs])
