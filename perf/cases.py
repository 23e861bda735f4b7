"""Measured cases of the gravity forward model and its adjoint on one MI355X.

Every case is one call (or one inversion step) of the public Python entry
points on a plan that the program keeps: ``Plan.eval``, ``Plan.adjoint``,
``Plan.direct`` and ``GravFMM``.  The sizes are those of the repository's own
workloads (README, tests, benchmark, serving loop): meshes of 16^3 to 256^3
cells, 1- and 2-point rules, stations above the mesh, all cell centres or
both, FP64 and mixed precision, one density or a batch, cell sources or
scattered ones.

Mixed-precision plans compute their M2L and near field in FP32, so a program
that chose one keeps its data and gradients as float32 tensors: those cases
convert the library's float64 buffers as such a program does.  FP64 cases
return the float64 results.

``exact`` evaluates the same sums in 64 bits with torch alone: cells,
centres and stations lie on lattices, so every sum is a convolution (FFT).
"""
import math

import torch

import paper_1107_5951_amd as G

DEV = "cuda"


def _case(name, kind, n, q=1, leaf=64, p=10, fp64=False, comps=1, batch=1, stations=1, centres=False, sources=0,
          points=0):
    c = {"kind": kind, "nx": n[0], "ny": n[1], "nz": n[2], "q": q, "leaf": leaf, "p": p, "fp64": fp64,
         "comps": comps, "batch": batch, "stations": stations, "centres": centres, "sources": sources,
         "points": points}
    return dict(c, name=name) if name else c


def listed():
    cube = lambda n: (n, n, n)
    return [
        # a survey of 1,024 stations over a 16^3 model, the smallest real call:
        # launches and latency count
        _case("survey16_fp64", "forward", cube(16), leaf=32, p=14, fp64=True, comps=3, stations=2),
        # serving requests (n in [32, 192], gz at n x n stations), odd and
        # ragged sizes, both directions and both rules
        _case("serve77_forward", "forward", cube(77)),
        _case("serve150_adjoint_q2", "adjoint", cube(150), q=2, leaf=512),
        # the field inside a 64^3 model with the 2-point rule, in both precisions
        _case("volume64_q2_mixed", "forward", cube(64), q=2, leaf=512, comps=3, stations=0, centres=True),
        _case("volume64_q2_fp64", "forward", cube(64), q=2, leaf=512, p=12, fp64=True, comps=3, stations=0,
              centres=True),
        # a box-shaped model with potential and field at its cells, gradient in FP64
        _case("box_adjoint_fp64", "adjoint", (120, 100, 70), p=12, fp64=True, comps=4, stations=0, centres=True),
        # the 256^3 model, field at all cells and 512^2 stations: forward,
        # gradient, and the FP64 reference solve
        _case("volume256_mixed", "forward", cube(256), comps=3, stations=2, centres=True),
        _case("volume256_adjoint", "adjoint", cube(256), comps=3, stations=2, centres=True),
        _case("volume256_fp64", "forward", cube(256), p=16, fp64=True, comps=3, stations=2, centres=True),
        # one iteration of an ensemble inversion: forward, misfit, gradient for
        # 32 density models of 128^3 cells
        _case("inversion128x32", "inversion", cube(128), batch=32, stations=2),
        # scattered sources with volumes (2 M points), gz at stations and
        # interior points
        _case("scattered2m", "forward", cube(128), batch=1, sources=2097152, points=65536, stations=2),
        # the summation method over the same mesh, the baseline users check against
        _case("direct48_fp64", "direct", cube(48), q=2, fp64=True, comps=3, stations=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges (cheaper than the largest of them)."""
    fam = rng.choice(["serve", "serve", "volume", "volume", "survey", "batch", "scattered", "direct"])
    if fam == "serve":
        q = rng.choice([1, 2])
        return _case(None, rng.choice(["forward", "adjoint"]), (_log(rng, 32, 192),) * 3, q=q, leaf=64 * q ** 3)
    if fam == "volume":
        fp64 = rng.random() < 0.4
        q = rng.choice([1, 2])
        m = _log(rng, 24, 128 if fp64 else 224)
        n = tuple(max(16, int(m * rng.uniform(0.6, 1.0))) for _ in range(3))
        return _case(None, rng.choice(["forward", "adjoint"]), n, q=q, leaf=64 * q ** 3,
                     p=rng.choice([12, 14, 16]) if fp64 else rng.choice([8, 10, 10]), fp64=fp64,
                     comps=rng.choice([1, 3, 3, 4]), stations=rng.choice([0, 1, 2]), centres=True)
    if fam == "survey":
        n = tuple(rng.randint(12, 48) for _ in range(3))
        return _case(None, rng.choice(["forward", "adjoint"]), n, leaf=rng.choice([32, 64]), p=rng.choice([12, 14]),
                     fp64=True, comps=rng.choice([1, 3]), stations=2)
    if fam == "batch":
        fp64 = rng.random() < 0.3
        return _case(None, "inversion", (_log(rng, 32, 112),) * 3, batch=rng.randint(2, 24), p=14 if fp64 else 10,
                     fp64=fp64, stations=rng.choice([1, 2]))
    if fam == "scattered":
        n = _log(rng, 24, 96)
        return _case(None, rng.choice(["forward", "adjoint"]), (n, n, n), comps=rng.choice([1, 3]),
                     sources=_log(rng, 20000, 800000), points=_log(rng, 1000, 30000), stations=1)
    return _case(None, "direct", (_log(rng, 16, 48),) * 3, q=rng.choice([1, 2]), fp64=rng.random() < 0.5, comps=3,
                 stations=1)


# --------------------------------------------------------------------- inputs
def _n(case):
    return case["nx"], case["ny"], case["nz"]


def _h(case):
    return 1.0 / max(_n(case))


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _uniform(g, shape, lo, hi):
    return lo + (hi - lo) * torch.rand(shape, dtype=torch.float64, device=DEV, generator=g)


def _density(case, seed):
    """Sums of Gaussian blobs sampled at the cell centres, a little noise on top: [batch, nz, ny, nx]."""
    g = _gen(seed)
    nx, ny, nz = _n(case)
    h = _h(case)
    ax = [(torch.arange(m, dtype=torch.float64, device=DEV) + 0.5) * h for m in (nx, ny, nz)]
    rho = torch.empty((case["batch"], nz, ny, nx), dtype=torch.float64, device=DEV)
    for b in range(case["batch"]):
        k = 8
        c = _uniform(g, (k, 3), 0.0, 1.0) * torch.tensor([nx * h, ny * h, nz * h], dtype=torch.float64, device=DEV)
        s = 0.5 / _uniform(g, (k, 1), 0.05, 0.2) ** 2
        a = torch.randn((k, 1), dtype=torch.float64, device=DEV, generator=g)
        ex, ey, ez = (torch.exp(-s * (ax[i][None, :] - c[:, i:i + 1]) ** 2) for i in range(3))
        zy = ((a * ez)[:, :, None] * ey[:, None, :]).reshape(k, nz * ny)
        rho[b] = (zy.t().contiguous() @ ex).reshape(nz, ny, nx)
    rho += _uniform(g, rho.shape, -0.01, 0.01)
    return rho


def _station_axes(case):
    """x and y of the k nx by k ny stations, and their height."""
    nx, ny, nz = _n(case)
    h, k = _h(case), case["stations"]
    x = (torch.arange(k * nx, dtype=torch.float64) + 0.5) * (h / k)
    y = (torch.arange(k * ny, dtype=torch.float64) + 0.5) * (h / k)
    return x, y, 1.1 * nz * h


def _points(case, seed):
    """Evaluation points of the plan: the stations, then interior points ([M, 3], host)."""
    pts = []
    if case["stations"]:
        x, y, z = _station_axes(case)
        yy, xx = torch.meshgrid(y, x, indexing="ij")
        pts.append(torch.stack([xx.reshape(-1), yy.reshape(-1), torch.full((xx.numel(),), z, dtype=torch.float64)], 1))
    if case["points"]:
        g = torch.Generator().manual_seed(int(seed) + 77)
        pts.append(torch.rand((case["points"], 3), dtype=torch.float64, generator=g)
                   * torch.tensor([m * _h(case) for m in _n(case)], dtype=torch.float64))
    return torch.cat(pts) if pts else None


def _sources(case, seed):
    """Scattered sources, denser towards the bottom, and their volumes (device)."""
    g = _gen(int(seed) + 55)
    u = torch.rand((case["sources"], 3), dtype=torch.float64, device=DEV, generator=g)
    u[:, 2] **= 1.5
    box = torch.tensor([m * _h(case) for m in _n(case)], dtype=torch.float64, device=DEV)
    vol = _uniform(g, (case["sources"],), 0.5, 1.5) * float(box.prod()) / case["sources"]
    return u * box, vol


def _targets(case):
    nx, ny, nz = _n(case)
    return case["stations"] ** 2 * nx * ny + case["points"] + (nx * ny * nz if case["centres"] else 0)


def prepare(case, seed):
    nx, ny, nz = _n(case)
    pts = _points(case, seed)
    src = vol = None
    if case["sources"]:
        src, vol = (t.cpu().numpy() for t in _sources(case, seed))
    plan = G.Plan(G.PlanSpec(n=(nx, ny, nz), h=_h(case), quad_order=case["q"],
                             points=None if pts is None else pts.numpy(), voxel_centres=case["centres"],
                             components=case["comps"], p=case["p"], leaf_size=case["leaf"],
                             precision=G.GRAV_FP64 if case["fp64"] else G.GRAV_MIXED, batch=case["batch"],
                             sources=src, source_volumes=vol))
    state = {"plan": plan, "kind": case["kind"], "out": torch.float64 if case["fp64"] else torch.float32}
    if case["kind"] == "adjoint":
        # data residuals, one per evaluation point and component
        state["resid"] = torch.randn(plan.out_shape, dtype=torch.float64, device=DEV, generator=_gen(seed))
    elif case["sources"]:
        # per-source densities
        state["rho"] = _uniform(_gen(seed), plan.rho_shape, 0.0, 2.0)
    else:
        state["rho"] = _density(case, seed)
    if case["kind"] == "inversion":
        state["rho"].requires_grad_(True)
        # observed data: of the size of the field, with noise
        state["data"] = torch.randn(plan.out_shape, dtype=torch.float64, device=DEV,
                                    generator=_gen(int(seed) + 1)).mul_(0.05).to(state["out"])
    return state


def run(state):
    plan, out = state["plan"], state["out"]
    if state["kind"] == "forward":
        return plan.eval(state["rho"]).to(out)
    if state["kind"] == "direct":
        return plan.direct(state["rho"]).to(out)
    if state["kind"] == "adjoint":
        return plan.adjoint(state["resid"]).to(out)
    rho = state["rho"]
    rho.grad = None
    field = G.GravFMM.apply(rho, plan)
    misfit = 0.5 * (field.to(out) - state["data"]).square().sum()
    misfit.backward()
    return {"field": field.detach().to(out), "misfit": misfit.detach(), "grad": rho.grad.to(out)}


def work(case):
    """The densities and the field (or residuals and gradient) once each in
    float64; and the operations of the method: per quadrature point and per
    target 2 p^2 a component (expansions), per leaf the translations, or 20
    per pair of the direct sum."""
    nx, ny, nz = _n(case)
    B, C, M = case["batch"], case["comps"], _targets(case)
    nsrc = case["sources"] or nx * ny * nz
    dirs = 2 if case["kind"] == "inversion" else 1
    bytes_ = 8 * B * (nsrc + M * C) * dirs
    if case["kind"] == "direct":
        return {"bytes": bytes_, "flops": 20.0 * M * nsrc * case["q"] ** 3 * B}
    p = case["p"]
    b = max(1, min(8, int(round((case["leaf"] / case["q"] ** 3) ** (1 / 3) - 0.17))))
    leaves = math.ceil(nx / b) * math.ceil(ny / b) * (math.ceil(nz / b) if case["centres"] or case["points"] else 1)
    flops = 2.0 * p * p * (nsrc + C * M) + 2.0 * p ** 4 * 27 * leaves
    return {"bytes": bytes_, "flops": flops * B * dirs}


# ---------------------------------------------------------------------- exact
def _pair(dx, dy, dz, q, comps):
    """Sum over a unit cell's quadrature points of the pair terms at offset
    (dx, dy, dz) from the cell centre, in cell units: the components wanted."""
    o = 0.5 / math.sqrt(3.0)
    offs = [(0.0, 0.0, 0.0)] if q == 1 else [(a, b, c) for a in (-o, o) for b in (-o, o) for c in (-o, o)]
    acc = None
    for a, b, c in offs:
        x, y, z = dx - a, dy - b, dz - c
        r2 = x * x + y * y + z * z
        ri = torch.where(r2 > 1e-20, r2.clamp_min(1e-20).rsqrt(), torch.zeros_like(r2)) / len(offs)
        ri3 = ri ** 3 * len(offs) ** 2
        t = {1: [z * ri3], 3: [x * ri3, y * ri3, z * ri3], 4: [ri, x * ri3, y * ri3, z * ri3]}[comps]
        acc = t if acc is None else [u + v for u, v in zip(acc, t)]
    return acc


def _scales(case):
    h = _h(case)
    return {1: [h], 3: [h, h, h], 4: [h * h, h, h, h]}[case["comps"]]


def _centre_kernels(case):
    """FFT of the centre-to-centre pair terms on the doubled mesh, one component after the other."""
    nx, ny, nz = _n(case)
    f = lambda m: torch.fft.fftfreq(2 * m, 1.0 / (2 * m), dtype=torch.float64, device=DEV).round()
    dz, dy, dx = (f(m).reshape(s) for m, s in ((nz, (-1, 1, 1)), (ny, (1, -1, 1)), (nx, (1, 1, -1))))
    z = torch.zeros((2 * nz, 2 * ny, 2 * nx), dtype=torch.float64, device=DEV)
    for k in range(case["comps"]):
        yield torch.fft.rfftn(_pair(dx + z, dy + z, dz + z, case["q"], case["comps"])[k])


def _station_kernels(case):
    """Per sub-lattice of stations and component: its slice of the k nx by k
    ny array and, per layer of cells, the FFT of the pair terms."""
    nx, ny, nz = _n(case)
    k = case["stations"]
    f = lambda m: torch.fft.fftfreq(2 * m, 1.0 / (2 * m), dtype=torch.float64, device=DEV).round()
    for sy in range(k):
        for sx in range(k):
            def layer(iz, sx=sx, sy=sy):
                dx = f(nx)[None, :] + ((sx + 0.5) / k - 0.5)
                dy = f(ny)[:, None] + ((sy + 0.5) / k - 0.5)
                dz = torch.full((), 1.1 * nz - (iz + 0.5), dtype=torch.float64, device=DEV)
                z = torch.zeros((2 * ny, 2 * nx), dtype=torch.float64, device=DEV)
                return torch.fft.rfft2(torch.stack(_pair(dx + z, dy + z, dz + z, case["q"], case["comps"])))
            yield (slice(sy, None, k), slice(sx, None, k)), layer


def _exact_forward(case, rho):
    nx, ny, nz = _n(case)
    B, C, k = case["batch"], case["comps"], case["stations"]
    sc = _scales(case)
    parts = []
    if k:
        st = torch.zeros((B, k * ny, k * nx, C), dtype=torch.float64, device=DEV)
        for (ry, rx), layer in _station_kernels(case):
            hat = torch.zeros((B, C, 2 * ny, nx + 1), dtype=torch.complex128, device=DEV)
            for iz in range(nz):
                hat += torch.fft.rfft2(rho[:, iz], s=(2 * ny, 2 * nx))[:, None] * layer(iz)[None]
            g = torch.fft.irfft2(hat, s=(2 * ny, 2 * nx))[:, :, :ny, :nx]
            for c in range(C):
                st[:, ry, rx, c] = g[:, c] * sc[c]
        parts.append(st.reshape(B, -1, C))
    if case["centres"]:
        g = torch.empty((B, nz * ny * nx, C), dtype=torch.float64, device=DEV)
        for c, kern in enumerate(_centre_kernels(case)):
            for b in range(B):
                hat = torch.fft.rfftn(rho[b], s=(2 * nz, 2 * ny, 2 * nx)) * kern
                g[b, :, c] = torch.fft.irfftn(hat, s=(2 * nz, 2 * ny, 2 * nx))[:nz, :ny, :nx].reshape(-1) * sc[c]
        parts.append(g)
    return torch.cat(parts, 1)


def _exact_adjoint(case, resid):
    nx, ny, nz = _n(case)
    B, C, k = case["batch"], case["comps"], case["stations"]
    sc = torch.tensor(_scales(case), dtype=torch.float64, device=DEV)
    drho = torch.zeros((B, nz, ny, nx), dtype=torch.float64, device=DEV)
    at = 0
    if k:
        at = k * k * nx * ny
        st = (resid[:, :at] * sc).reshape(B, k * ny, k * nx, C)
        for (ry, rx), layer in _station_kernels(case):
            hat = torch.fft.rfft2(st[:, ry, rx].permute(0, 3, 1, 2).contiguous(), s=(2 * ny, 2 * nx))
            for iz in range(nz):
                g = (hat * layer(iz).conj()[None]).sum(1)
                drho[:, iz] += torch.fft.irfft2(g, s=(2 * ny, 2 * nx))[:, :ny, :nx]
    if case["centres"]:
        r = (resid[:, at:] * sc).reshape(B, nz, ny, nx, C)
        for c, kern in enumerate(_centre_kernels(case)):
            for b in range(B):
                hat = torch.fft.rfftn(r[b, ..., c].contiguous(), s=(2 * nz, 2 * ny, 2 * nx)) * kern.conj()
                drho[b] += torch.fft.irfftn(hat, s=(2 * nz, 2 * ny, 2 * nx))[:nz, :ny, :nx]
    return drho


def _exact_scattered(case, seed, value):
    """Plain sums over the pairs of scattered sources and points, in blocks."""
    src, vol = _sources(case, seed)
    pts = _points(case, seed).to(DEV)
    h, C = _h(case), case["comps"]
    adj = case["kind"] == "adjoint"
    out = torch.zeros((src.shape[0],) if adj else (pts.shape[0], C), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 26) // src.shape[0])
    for i in range(0, pts.shape[0], step):
        t = pts[i:i + step]
        d = [t[:, a:a + 1] - src[None, :, a] for a in range(3)]
        r2 = d[0] ** 2 + d[1] ** 2 + d[2] ** 2
        ri3 = torch.where(r2 > (1e-10 * h) ** 2, r2.rsqrt() ** 3, torch.zeros_like(r2))
        for c, a in enumerate([2] if C == 1 else [0, 1, 2]):
            if adj:
                out += (value[0, i:i + step, c] @ (d[a] * ri3)) * vol
            else:
                out[i:i + step, c] = (d[a] * ri3) @ (value[0] * vol)
    return out[None]


def exact(case, seed):
    if case["sources"] and case["sources"] * _targets(case) > 2e10:
        return None  # minutes of plain summation
    nx, ny, nz = _n(case)
    fwd_shape = (case["batch"], _targets(case), case["comps"])
    value = None
    if case["kind"] == "adjoint":
        value = torch.randn(fwd_shape, dtype=torch.float64, device=DEV, generator=_gen(seed))
    elif case["sources"]:
        value = _uniform(_gen(seed), (1, case["sources"]), 0.0, 2.0)
    if case["sources"]:
        return _exact_scattered(case, seed, value)
    if case["kind"] == "adjoint":
        return _exact_adjoint(case, value)
    rho = _density(case, seed)
    field = _exact_forward(case, rho)
    if case["kind"] != "inversion":
        # Plan.eval drops the batch dimension only for [nz, ny, nx] densities
        return field
    data = torch.randn(fwd_shape, dtype=torch.float64, device=DEV, generator=_gen(int(seed) + 1)).mul_(0.05)
    data = data.to(torch.float64 if case["fp64"] else torch.float32).double()
    return {"field": field, "misfit": 0.5 * (field - data).square().sum(),
            "grad": _exact_adjoint(case, field - data)}
