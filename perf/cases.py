"""What a user of this library has it do, as cases that can be timed and checked.

A case is one observation (stations in a disc, all baselines or some of them, timesteps of
earth rotation, channels over 140-170 MHz) with its imaging geometry, and one call on it:

  grid      plan.grid: visibilities -> w-layer grids
  degrid    plan.degrid: grids of a lattice point-source sky -> visibilities
  train     autograd.degrid and its backward: visibilities and the gradient of the grid
  sky       autograd.predict_vis: image -> visibilities (w-stacked prediction, degridding)
  invert    plan.invert: w-layer grids -> image
  jobs      Executor.execute: gridding and degridding of several plans in shared launches

Sizes run from the CPU-sized observation (16 stations, 3840 visibilities) over a served
mix's jobs to the MWA-like one (128 stations, 46.8M visibilities, 8000^2 grid).
"""
import math

import numpy as np
import torch

import paper_2502_17789_amd as aidg
from paper_2502_17789_amd import autograd

C = 299792458.0
ARCSEC = math.pi / 648000.0


def _case(name, kind, **kw):
    c = dict(kind=kind, stations=16, diameter=5000.0, times=8, dt=2.0, channels=4, every=1, N=1024, L=32, ha=0.0,
             fp64=False, stokes=False, fold=False, inverse=False, table=False, jobs=1, sources=8)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        _case("grid_small", "grid", diameter=1000.0, N=512, table=True),
        _case("degrid_small", "degrid", diameter=1000.0, N=512),
        _case("grid_odd", "grid", stations=23, diameter=1500.0, times=11, channels=13, N=1000, L=64, table=True),
        _case("degrid_sparse", "degrid", stations=48, times=12, channels=3, every=32, N=2048, L=96),
        _case("train_medium", "train", stations=64, times=30, channels=48, N=4096, L=64),
        _case("grid_stokes_fold", "grid", stations=72, times=16, channels=96, N=4096, L=32, ha=0.4, stokes=True,
              fold=True, inverse=True),
        _case("degrid_fp64", "degrid", stations=40, times=16, channels=32, N=2048, L=96, fp64=True),
        _case("jobs_mixed", "jobs", stations=40, times=6, channels=16, N=1024, L=32, jobs=8),
        _case("sky_2048", "sky", stations=32, times=20, channels=32, N=2048, L=64, ha=0.3),
        _case("invert_8000", "invert", stations=128, times=4, channels=8, N=8000, L=96, ha=0.03, fold=True),
        _case("grid_mwa", "grid", stations=128, times=60, channels=96, N=8000, L=96),
        _case("degrid_mwa", "degrid", stations=128, times=60, channels=96, N=8000, L=96),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["grid", "grid", "degrid", "degrid", "train", "sky", "invert", "jobs"])
    L = rng.choice([32, 64, 96])
    N = rng.choice([512, 1000, 1024, 2048, 4096, 8000]) if kind != "sky" else rng.choice([512, 1024, 2048, 4096])
    if kind == "sky":
        L = rng.choice([32, 64])
    case = _case(None, kind, stations=log(8, 128), diameter=rng.choice([1000.0, 5000.0]), times=log(1, 60),
                 channels=log(1, 96), N=N, L=L, ha=rng.choice([0.0, 0.0, 0.2]), stokes=rng.random() < 0.2,
                 fold=rng.random() < 0.3, sources=rng.randint(1, 12))
    if kind in ("grid", "degrid"):
        case["fp64"] = rng.random() < 0.2 and N <= 4096
        case["every"] = rng.choice([1, 1, 1, 8])
        case["channels"] = max(1, case["channels"] // (4 if case["every"] > 1 else 1))
        case["inverse"] = kind == "grid" and rng.random() < 0.25
    if kind == "jobs":
        case.update(jobs=rng.randint(2, 12), stations=log(16, 64), times=log(1, 8), N=min(N, 2048), ha=0.0)
    if kind == "invert":
        case.update(ha=rng.choice([0.0, 0.02]), times=2, channels=2)
    if N > 4096:
        case.update(ha=min(case["ha"], 0.02))
    most = 4e6 if case["fp64"] else 16e6
    while _visibilities(case) > most:  # no drawn case costs more than the MWA-like one
        case["times"] = max(1, case["times"] // 2)
        case["stations"] = max(8, int(case["stations"] * 0.8))
    return case


def _visibilities(case):
    nbl = case["stations"] * (case["stations"] - 1) // 2
    return nbl * case["times"] * case["channels"] * case["jobs"]


# ------------------------------------------------------------------ the observation


def _observation(case):
    """Stations uniform in a disc at latitude -26.7 deg, phase centre at -27 deg.
    The array is the case's own: seeds change the sky, the A-terms and the data."""
    rng = np.random.default_rng(case["stations"])
    n, nt = case["stations"], case["times"]
    r, th = 0.5 * case["diameter"] * np.sqrt(rng.random(n)), 2 * math.pi * rng.random(n)
    east, north = r * np.cos(th), r * np.sin(th)
    lat, dec = math.radians(-26.7), math.radians(-27.0)
    xyz = np.stack([-math.sin(lat) * north, east, math.cos(lat) * north])
    p, q = np.triu_indices(n, k=1)
    bl = np.stack([p, q], axis=1).astype(np.int32)
    bx, by, bz = (xyz[:, q] - xyz[:, p])[:, :, None]
    h = case["ha"] + (np.arange(nt) - 0.5 * (nt - 1)) * case["dt"] * 7.2921159e-5
    sh, ch, sd, cd = np.sin(h), np.cos(h), math.sin(dec), math.cos(dec)
    uvw = np.stack([sh * bx + ch * by, -sd * ch * bx + sd * sh * by + cd * bz,
                    cd * ch * bx - cd * sh * by + sd * bz], axis=-1)
    nc = case["channels"] * case["every"]
    freqs = (140e6 + (np.arange(nc) + 0.5) * 30e6 / nc)[::case["every"]]
    umax = max(float(np.abs(uvw[..., :2]).max()) * freqs[-1] / C, 1.0)
    return bl, np.ascontiguousarray(uvw), freqs, umax


def _geometry(case, umax):
    N, L = case["N"], case["L"]
    K = L // 4
    # Nyquist with the window of the outermost subgrid on the grid, 15 arcsec or finer
    dl = min(15.0 * ARCSEC * max(1.0, 2000.0 / N), (0.5 - (K + 2.0) / N) * 0.95 / umax, 0.6 / N)
    return aidg.Geometry(N, L, K, dl, aterm_interval=8, w_step=-1.0 if case["table"] else 0.0,
                         precision=aidg.FP64 if case["fp64"] else aidg.FP32, stokes_i=int(case["stokes"]),
                         w_fold=int(case["fold"]), aterm_mode=int(case["inverse"]))


def _layers(case, geo, uvw, freqs):
    """The w-layers of the automatic spacing 2 w_max, w_max = K / (4 FOV rho), rho = max |grad n|;
    folded rows lie at w >= 0 on odd multiples of half the spacing."""
    fov = geo.grid_size * geo.pixel_scale
    r = fov / math.sqrt(2.0)
    step = 2 * geo.kernel_support / (4 * fov * r / math.sqrt(1 - r * r))
    w = uvw[..., 2][:, :, None] * freqs / C
    j = np.floor(np.abs(w) / step) if case["fold"] else np.rint(w / step)
    return (np.arange(int(j.min()), int(j.max()) + 1) + (0.5 if case["fold"] else 0.0)) * step


def _dtype(case):
    return torch.complex128 if case["fp64"] else torch.complex64


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _noise(shape, g, dtype):
    return torch.randn(shape, dtype=dtype, device="cuda", generator=g)


def _aterms(case, geo, seed):
    """Beam times a smooth phase screen per interval and station, with a little leakage."""
    n_int, n, L = -(-case["times"] // 8), case["stations"], case["L"]
    g = _generator(seed + 1000)
    coarse = torch.randn((n_int * n, 1, 8, 8), device="cuda", generator=g)
    phi = torch.nn.functional.interpolate(coarse, size=(L, L), mode="bilinear", align_corners=True)
    c = (torch.arange(L, device="cuda") - L // 2) * (geo.grid_size * geo.pixel_scale / L)
    sig = math.radians(25.0) / 2.3548
    beam = torch.exp(-0.5 * (c[:, None] ** 2 + c[None, :] ** 2) / sig ** 2)
    e = torch.polar(beam.expand(n_int * n, L, L).contiguous(), phi[:, 0]).reshape(n_int, n, L, L)
    gain = 1 + 0.1 * _noise((2, n_int, n, 1, 1), g, torch.complex64)
    leak = 0.05 * _noise((2, n_int, n, 1, 1), g, torch.complex64)
    A = torch.stack([e * gain[0], e * leak[0], e * leak[1], e * gain[1]], dim=-1)
    return A.to(_dtype(case)).contiguous()


def _axis_taper(n, beta):
    f = (np.arange(n) - n // 2) / n
    return np.i0(beta * np.sqrt(np.maximum(0.0, 1.0 - 4.0 * f * f))) / np.i0(beta)


def _sky(case, geo, seed):
    """Point sources on subgrid-lattice pixels of the taper's main lobe: pixel indices,
    direction cosines, n - 1 and Hermitian brightness matrices [n, 4]."""
    rng = np.random.default_rng(seed + 2000)
    n, L = case["sources"], case["L"]
    xs, ys = rng.integers(L // 4, 3 * L // 4 + 1, (2, n))
    step = geo.grid_size * geo.pixel_scale / L
    l, m = (xs - L // 2) * step, (ys - L // 2) * step
    flux = np.exp(rng.uniform(math.log(0.1), math.log(10.0), n))
    q, u, v = rng.uniform(-0.1, 0.1, (3, n)) * flux * (0.0 if case["stokes"] else 1.0)
    B = np.stack([flux + q, u + 1j * v, u - 1j * v, flux - q], axis=1)
    return xs, ys, l, m, np.sqrt(1 - l * l - m * m) - 1, B


def _sky_grid(case, geo, w0s, seed):
    """Grid of the sky: plane waves scaled so that degridding returns the sources' visibilities."""
    xs, ys, l, m, n1, B = _sky(case, geo, seed)
    N, L = geo.grid_size, geo.subgrid_size
    t = _axis_taper(L, math.pi * geo.kernel_support / 4)
    cell = (np.arange(N) - N // 2) / (N * geo.pixel_scale)
    dt = _dtype(case)
    pol = [0] if case["stokes"] else range(4)
    G = torch.empty((len(w0s), len(pol), N, N), dtype=dt, device="cuda")
    for w, w0 in enumerate(w0s):
        ev = torch.from_numpy(np.exp(-2j * np.pi * np.outer(cell, m))).cuda()
        eu = torch.from_numpy(np.exp(-2j * np.pi * np.outer(cell, l))).cuda()
        for j, p in enumerate(pol):
            amp = B[:, p] * np.exp(-2j * np.pi * w0 * n1) / (L * L * t[xs] * t[ys])
            G[w, j] = ((ev * torch.from_numpy(amp).cuda()) @ eu.T.contiguous()).to(dt)
    return G


def _sky_image(case, geo, seed):
    """Image of the sky (the lattice pixels are image pixels where L divides N)."""
    xs, ys, _, _, _, B = _sky(case, geo, seed)
    N, L = geo.grid_size, geo.subgrid_size
    image = torch.zeros((1 if case["stokes"] else 4, N, N), dtype=_dtype(case), device="cuda")
    for k in range(len(xs)):
        for p in range(image.shape[0]):
            image[p, int(ys[k]) * (N // L), int(xs[k]) * (N // L)] += complex(B[k, p])
    return image


def _tables(case, geo, bl, uvw, freqs):
    """A program's own sub-tables: halved in time or channels until their uv extent fits."""
    N, L, K = geo.grid_size, geo.subgrid_size, geo.kernel_support
    fov, rows = N * geo.pixel_scale, []
    nt, nc = uvw.shape[1], len(freqs)
    for b in range(len(bl)):
        todo = [(t, min(8, nt - t), 0, nc) for t in range(0, nt, 8)]
        while todo:
            t0, n, c0, k = todo.pop()
            ends = uvw[b, t0:t0 + n, None, :2] * freqs[[c0, c0 + k - 1]][None, :, None] / C * fov
            lo, hi = ends.min(axis=(0, 1)), ends.max(axis=(0, 1))
            if max(hi - lo) > L - K - 2 and n * k > 1:
                split = [(t0, n, c0, k // 2), (t0, n, c0 + k // 2, k - k // 2)] if k > 1 else \
                    [(t0, n // 2, c0, k), (t0 + n // 2, n - n // 2, c0, k)]
                todo += split
                continue
            U0, V0 = np.clip(np.rint(0.5 * (lo + hi)).astype(int) + N // 2, L // 2, N - L // 2)
            rows.append((b, bl[b, 0], bl[b, 1], t0, n, c0, k, U0, V0, 0, t0 // 8, 0, 0.0, (b * nt + t0) * nc + c0))
    return np.array(rows, dtype=aidg.SUBGRID_DTYPE)


# ------------------------------------------------------------------ one case


def _jobs(case):
    """The jobs of a mixed launch: every other one a degridding, of uneven sizes."""
    return [dict(case, kind="grid" if j % 2 == 0 else "degrid", jobs=1, stations=max(8, case["stations"] - 3 * j),
                 times=1 + (j * 5) % case["times"], L=(32, 64, 96)[(j + case["L"] // 32 - 1) % 3])
            for j in range(case["jobs"])]


def prepare(case, seed):
    if case["kind"] == "jobs":
        items = [prepare(one, seed + 17 * j) for j, one in enumerate(_jobs(case))]
        return {"kind": "jobs", "items": items, "executor": aidg.Executor(256 << 20)}
    bl, uvw, freqs, umax = _observation(case)
    geo = _geometry(case, umax)
    table = _tables(case, geo, bl, uvw, freqs) if case["table"] else None
    plan = aidg.Plan(geo, case["stations"], bl, uvw, freqs, _aterms(case, geo, seed), table=table)
    s = {"kind": case["kind"], "plan": plan}
    if case["kind"] == "grid":
        s["in"] = _noise(plan.vis_shape(), _generator(seed), _dtype(case))
    elif case["kind"] == "invert":
        s["in"] = _noise(plan.grid_shape(), _generator(seed), _dtype(case))
    elif case["kind"] == "sky":
        s["in"] = _sky_image(case, geo, seed)
    else:
        s["in"] = _sky_grid(case, geo, plan.wlayers(), seed)
    if case["kind"] == "train":
        s["in"].requires_grad_(True)
        s["gradient"] = _noise(plan.vis_shape(), _generator(seed), _dtype(case))
    return s


def run(state):
    kind = state["kind"]
    if kind == "jobs":
        work, outs = [], []
        for s in state["items"]:
            p = s["plan"]
            grid = s["kind"] == "grid"
            out = torch.zeros(p.grid_shape(), dtype=s["in"].dtype, device="cuda") if grid else \
                torch.empty(p.vis_shape(), dtype=s["in"].dtype, device="cuda")
            work.append((p, aidg.DIR_GRID if grid else aidg.DIR_DEGRID, s["in"], out, 0, p.info["n_subgrids"]))
            outs.append(out)
        state["executor"].execute(work)
        return outs
    plan, x = state["plan"], state["in"]
    if kind == "grid":
        return plan.grid(x)
    if kind == "degrid":
        return plan.degrid(x)
    if kind == "invert":
        return plan.invert(x)
    if kind == "sky":
        return autograd.predict_vis(x, plan)
    vis = autograd.degrid(x, plan)
    grad, = torch.autograd.grad(vis, x, state["gradient"])
    return {"vis": vis.detach(), "grad": grad}


def work(case):
    """Bytes: inputs read once and outputs written once (visibilities, A-terms, grids, images).
    Operations: 16 multiply-adds per visibility and subgrid pixel (the 2x2 complex sum), and
    5 N log2 N for each of the image level's row transforms."""
    if case["kind"] == "jobs":
        total = {"bytes": 0.0, "flops": 0.0}
        for one in _jobs(case):
            for key, value in work(one).items():
                total[key] += value
        return total
    e = 16 if case["fp64"] else 8
    pols = 1 if case["stokes"] else 4
    N, L, nv = case["N"], case["L"], _visibilities(case)
    layers = 1
    if not case["table"]:
        bl, uvw, freqs, umax = _observation(case)
        layers = len(_layers(case, _geometry(case, umax), uvw, freqs))
    grid, image = layers * pols * N * N * e, pols * N * N * e
    aterms = -(-case["times"] // 8) * case["stations"] * L * L * 4 * e
    passes = {"grid": 1, "degrid": 1, "sky": 1, "train": 2, "invert": 0}[case["kind"]]
    b = passes * (nv * 4 * e + aterms + grid)
    f = passes * 32.0 * nv * L * L
    if case["kind"] in ("sky", "invert"):
        b, f = b + grid + image, f + layers * pols * 2 * N * 5.0 * N * math.log2(N)
    return {"bytes": float(b), "flops": float(f)}


# ------------------------------------------------------------------ exact values


def _exact_vis(case, seed):
    """Visibilities of the sky by the measurement equation, V = sum_s A_p B_s A_q^H e(-phase)."""
    bl, uvw, freqs, umax = _observation(case)
    geo = _geometry(case, umax)
    xs, ys, l, m, n1, B = _sky(case, geo, seed)
    A = _aterms(case, geo, seed)[:, :, ys, xs, :].to(torch.complex128)  # [int, st, s, 4]
    A = A.reshape(A.shape[:3] + (2, 2))
    Bm = torch.from_numpy(B.reshape(-1, 2, 2)).cuda()
    lmn = [torch.from_numpy(v).cuda() for v in (l, m, n1)]
    fc = torch.from_numpy(freqs / C).cuda()
    nbl, nt, nc = len(bl), uvw.shape[1], len(freqs)
    out = torch.zeros((nbl, nt, nc, 4), dtype=torch.complex128, device="cuda")
    at = torch.arange(nt, device="cuda") // 8
    for b0 in range(0, nbl, 256):
        u = torch.from_numpy(uvw[b0:b0 + 256]).cuda()
        p, q = (torch.from_numpy(bl[b0:b0 + 256, i].astype(np.int64)).cuda() for i in (0, 1))
        for s in range(len(xs)):
            Ap, Aq = A[:, p, s], A[:, q, s]  # [int, b, 2, 2]
            AB = (Ap[..., :, :, None] * Bm[s]).sum(-2)
            J = (AB[..., :, None, :] * Aq[..., None, :, :].conj()).sum(-1).reshape(AB.shape[:2] + (4,))
            turns = (u[..., 0] * lmn[0][s] + u[..., 1] * lmn[1][s] + u[..., 2] * lmn[2][s])[:, :, None] * fc
            turns = turns - torch.round(turns)
            ph = torch.polar(torch.ones_like(turns), -2 * math.pi * turns)
            out[b0:b0 + 256] += ph[..., None] * J[at].transpose(0, 1)[:, :, None, :]
    return out


def _exact_grid(case, seed):
    """The grid of the program's own sub-tables: every subgrid's direct phasor sum, Jones
    correction, taper, centred transform and addition, in 64 bits."""
    bl, uvw, freqs, umax = _observation(case)
    geo = _geometry(case, umax)
    N, L = geo.grid_size, geo.subgrid_size
    table = _tables(case, geo, bl, uvw, freqs)
    A = _aterms(case, geo, seed).to(torch.complex128).reshape(-1, case["stations"], L * L, 2, 2)
    vis = _noise((len(bl), uvw.shape[1], len(freqs), 4), _generator(seed), _dtype(case)).to(torch.complex128)
    fov = N * geo.pixel_scale
    c = torch.from_numpy((np.arange(L) - L // 2) * (fov / L)).cuda()
    l, m = c[None, :].expand(L, L).reshape(-1), c[:, None].expand(L, L).reshape(-1)
    n1 = torch.sqrt(1 - l * l - m * m) - 1
    t = torch.from_numpy(_axis_taper(L, math.pi * geo.kernel_support / 4)).cuda()
    T = (t[:, None] * t[None, :]).reshape(-1)
    duvw, fc = torch.from_numpy(uvw).cuda(), torch.from_numpy(freqs / C).cuda()
    G = torch.zeros((1, 4, N, N), dtype=torch.complex128, device="cuda")
    for s in table:
        b, t0, n, c0, k, U0, V0 = (int(s[f]) for f in ("bl", "t0", "nt", "c0", "nc", "U0", "V0"))
        w = (duvw[b, t0:t0 + n, None, :] * fc[None, c0:c0 + k, None]).reshape(-1, 3)
        turns = (w[:, 0:1] - (U0 - N // 2) / fov) * l + (w[:, 1:2] - (V0 - N // 2) / fov) * m + w[:, 2:3] * n1
        turns = turns - torch.round(turns)
        ph = torch.polar(torch.ones_like(turns), 2 * math.pi * turns)
        S = (ph.T.contiguous() @ vis[b, t0:t0 + n, c0:c0 + k].reshape(-1, 4)).reshape(-1, 2, 2)
        Ap, Aq = A[int(s["aint"]), int(s["st1"])], A[int(s["aint"]), int(s["st2"])]
        AS = (Ap.conj()[:, :, :, None] * S[:, :, None, :]).sum(1)  # A_p^H S
        S = (AS[:, :, :, None] * Aq[:, None, :, :]).sum(2)
        S = (S.reshape(-1, 4) * T[:, None]).T.reshape(4, L, L)
        F = torch.fft.fftshift(torch.fft.fft2(torch.fft.ifftshift(S, dim=(1, 2))), dim=(1, 2))
        G[0, :, V0 - L // 2:V0 + L // 2, U0 - L // 2:U0 + L // 2] += F
    return G


def _exact_image(case, seed):
    """The w-stacked image of the grids by 64-bit transforms."""
    bl, uvw, freqs, umax = _observation(case)
    geo = _geometry(case, umax)
    N, L, K = geo.grid_size, geo.subgrid_size, geo.kernel_support
    w0s = _layers(case, geo, uvw, freqs)
    pol = 1 if case["stokes"] else 4
    G = _noise((len(w0s), pol, N, N), _generator(seed), _dtype(case))
    c = torch.from_numpy((np.arange(N) - N // 2) * geo.pixel_scale).cuda()
    r2 = c[None, :] ** 2 + c[:, None] ** 2
    n1 = -r2 / (1 + torch.sqrt(1 - r2))
    t = torch.from_numpy(_axis_taper(N, math.pi * K / 4)).cuda()
    image = torch.zeros((pol, N, N), dtype=torch.complex128, device="cuda")
    for k, w0 in enumerate(w0s):
        phase = torch.polar(torch.ones_like(n1), 2 * math.pi * w0 * n1)
        for p in range(pol):
            F = torch.fft.ifft2(torch.fft.ifftshift(G[k, p].to(torch.complex128)), norm="forward")
            image[p] += torch.fft.fftshift(F) * phase
    return image / (L * L * t[:, None] * t[None, :])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("degrid", "sky"):
        return _exact_vis(case, seed)
    if kind == "train":
        return {"vis": _exact_vis(case, seed), "grad": None}
    if kind == "grid" and case["table"]:
        return _exact_grid(case, seed)
    if kind == "invert":
        return _exact_image(case, seed)
    return None  # the grid of a partition that the library chose
