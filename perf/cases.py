"""The work a user of this framework has it do, as measurable cases.

A case names an operation, a geometry and a slice count; `prepare` makes what a
reconstruction program holds before the call (projections or images in HBM, the
geometry object, output and workspace buffers), `run` is one call of a public
entry point on them, `work` the bytes and operations the call cannot do without,
and `exact` its result in 64 bits from plain torch.

Operations:
    reconstruct  fbp_reconstruct of a slice or a stack (parallel or fan beam)
    batch        fbp_reconstruct_batch of slices of mixed sizes (parallel beam)
    project      fbp_project, the adjoint used by iterative methods (parallel or fan beam)
    cone         fbp_cone_reconstruct (FDK) of a volume
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2109_02174_amd as fbp

GOLDEN = math.pi * (math.sqrt(5.0) - 1.0) / 2.0

# Largest number of pixel-angle updates of a drawn call: that of the largest listed stack.
MOST_UPDATES = 64 * 512 * 512 * 720


def diagonal_bins(side: int) -> int:
    """Bins of unit width that cover the image diagonal, and a margin of two."""
    return int(math.ceil(math.sqrt(2.0) * side)) + 2


def fan_bins(side: int, R: float) -> int:
    """Bins of a flat detector through the centre that see the whole image from distance R."""
    r = side / math.sqrt(2.0)
    return int(math.ceil(2.0 * R * r / math.sqrt(R * R - r * r))) + 2


def parallel(name, side, angles, bins, slices, op="reconstruct", precision="fp32", filter="ramlak", list="uniform",
             weighting="uniform", dt=1.0):
    c = dict(op=op, side=side, angles=angles, bins=bins, dt=dt, slices=slices, source=0.0, list=list)
    if op == "reconstruct":
        c.update(precision=precision, filter=filter)
    if op != "batch":
        c.update(weighting=weighting)
    return dict(c, name=name) if name else c


def fan(name, side, angles, bins, source, slices, op="reconstruct", precision="fp32", filter="ramlak", dt=1.0):
    c = dict(op=op, side=side, angles=angles, bins=bins, dt=dt, slices=slices, source=float(source), list="uniform",
             weighting="uniform")
    if op == "reconstruct":
        c.update(precision=precision, filter=filter)
    return dict(c, name=name) if name else c


def cone(name, side, depth, views, rows, columns, source, filter="ramlak"):
    c = dict(op="cone", side=side, depth=depth, angles=views, rows=rows, bins=columns, source=float(source),
             filter=filter)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: one 128^2 preview slice as it arrives; launches and latency count.
        parallel("slice_128", 128, 180, 183, 1),
        # The ordinary call: one 512^2 slice at full angular sampling, a request at a time.
        parallel("slice_512", 512, 720, 725, 1),
        # Throughput: a volume's slices of one geometry in one call.
        parallel("stack_512", 512, 720, 725, 64),
        # A volume at reduced filter precision, odd image side and detector.
        parallel("stack_511_bf16", 511, 600, 725, 24, precision="bf16"),
        # A dynamic acquisition: golden-angle views (no symmetry in the list), gap weights, Hann kernel.
        parallel("slice_golden", 400, 601, 568, 1, filter="hann", list="golden", weighting="angle-gaps"),
        # One large slice through the FFT filter, which is there for long detectors.
        parallel("slice_1024_fft", 1024, 1440, 1451, 1, precision="fft"),
        # Requests of mixed sizes gathered into one call, as the serving loop sends them.
        dict(op="batch", name="batch_mixed", slices=48, mix=4),
        # Fan beam: one slice, and a stack with ragged sides.
        fan("fan_slice", 512, 720, 801, 1024.0, 1),
        fan("fan_stack", 365, 540, 611, 640.0, 12, filter="hann"),
        # Forward projection of the current estimate in an iterative method, parallel and fan beam.
        parallel("project_slice", 512, 720, 725, 1, op="project"),
        fan("project_fan", 512, 720, 801, 1024.0, 2, op="project"),
        # A cone-beam volume.
        cone("cone_256", 256, 256, 360, 256, 384, 512.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("slice", "slice", "stack", "stack", "list", "batch", "fan", "fan", "project", "project_fan", "cone"))
    if kind == "batch":
        return dict(op="batch", slices=_log_int(rng, 4, 48), mix=rng.randrange(1 << 20))
    if kind == "cone":
        side = _log_int(rng, 32, 256)
        depth = rng.randint(max(8, side // 3), side)
        source = side * rng.uniform(1.6, 3.0)
        views = _log_int(rng, 60, 360)
        columns = fan_bins(side, source)
        rows = int(math.ceil(depth * source / (source - side / math.sqrt(2.0)))) + 2
        if rng.random() < 0.5:
            columns = (columns + 3) // 4 * 4
        return cone(None, side, depth, views, rows, columns, round(source, 2), rng.choice(("ramlak", "hann")))
    side, angles = _log_int(rng, 64, 1024), _log_int(rng, 60, 1440)
    if rng.random() < 0.6:
        angles = (angles + 3) // 4 * 4
    slices = 1 if kind in ("slice", "list") else _log_int(rng, 2, 64) if kind == "stack" else _log_int(rng, 1, 16)
    most = MOST_UPDATES if kind in ("slice", "list", "stack") else MOST_UPDATES // 4 if kind == "fan" else MOST_UPDATES // 16
    while side * side * angles * slices > most:
        if slices > 1:
            slices = (slices + 1) // 2
        else:
            side = side * 3 // 4
    filter = rng.choice(("ramlak", "ramlak", "ramlak", "hann", "shepp-logan"))
    precision = rng.choice(("fp32", "fp32", "fp32", "bf16", "fp16", "fft"))
    if precision in ("bf16", "fp16"):
        filter = "ramlak"                   # the kernel whose rounded taps keep the exact mean response
    if kind in ("fan", "project_fan"):
        source = round(side * rng.uniform(1.5, 4.0), 2)
        return fan(None, side, angles, fan_bins(side, source), source, slices,
                   op="project" if kind == "project_fan" else "reconstruct", precision=precision, filter=filter)
    dt = rng.choice((1.0, 1.0, 1.0, 0.75, 1.25))
    bins = max(1, int(diagonal_bins(side) / dt))
    if rng.random() < 0.2:
        bins = max(1, int(bins * 0.8))      # a detector shorter than the image diagonal
    uneven = kind == "list" and rng.random() < 0.6
    if kind == "list" and not uneven:
        angles |= 1                         # even spacing, odd count: no quarter turns
    return parallel(None, side, angles, bins, slices, op="project" if kind == "project" else "reconstruct",
                    precision=precision, filter=filter, list="golden" if uneven else "uniform",
                    weighting="angle-gaps" if uneven else "uniform", dt=dt)


# ---------------------------------------------------------------- inputs

def _angles(case):
    K = case["angles"]
    if case["list"] == "golden":
        return np.mod(np.arange(K, dtype=np.float64) * GOLDEN, math.pi)
    return np.arange(K, dtype=np.float64) * ((2.0 if case["source"] > 0 else 1.0) * math.pi / K)


def _geometry(case):
    return fbp.Geometry(case["angles"], case["bins"], case["side"], case["dt"], _angles(case),
                        filter=case.get("filter", "ramlak"), weighting=case["weighting"],
                        source_distance=case["source"])


def _cone_geometry(case):
    return fbp.ConeGeometry(case["angles"], case["bins"], case["rows"], case["side"], case["depth"], case["source"],
                            filter=case["filter"])


def _batch_geometries(case):
    """Sides, angle counts and detectors of the mixed batch, by its own generator."""
    rng = np.random.Generator(np.random.PCG64(case["mix"]))
    out = []
    for _ in range(case["slices"]):
        side = int(rng.choice((256, 384, 512, 1024)))
        out.append((side, int(rng.choice((360, 720, 1440))), diagonal_bins(side)))
    return out


def _ellipses(seed, slices, n=8):
    """Random ellipses [slices][n][6] in units of half the image: centre, semi-axes, rotation, density."""
    rng = np.random.Generator(np.random.PCG64(seed))
    lo = np.array([-0.6, -0.6, 0.05, 0.05, 0.0, -0.5])
    hi = np.array([0.6, 0.6, 0.4, 0.4, math.pi, 1.0])
    return rng.uniform(lo, hi, size=(slices, n, 6))


def _sinograms(case, seed, device="cuda"):
    """Line integrals of the ellipses (pixel units, evaluated on the GPU) and 0.5 % of noise."""
    B, K, D, N = case["slices"], case["angles"], case["bins"], case["side"]
    ang = torch.as_tensor(_angles(case), device=device).view(1, K, 1)
    t = ((torch.arange(D, device=device, dtype=torch.float64) - 0.5 * (D - 1)) * case["dt"]).view(1, 1, D)
    R = case["source"]
    if R > 0:
        ang = ang + 0.5 * math.pi - torch.atan(t / R)
        t = R * t / torch.sqrt(R * R + t * t)
    ang, t = ang.float(), t.float()
    e = torch.as_tensor(_ellipses(seed, B), device=device, dtype=torch.float32)
    h = 0.5 * N
    sino = torch.zeros((B, K, D), device=device, dtype=torch.float32)
    ca, sa = torch.cos(ang), torch.sin(ang)
    for i in range(e.shape[1]):
        x0, y0, a, b, phi, rho = (e[:, i, q].view(B, 1, 1) for q in range(6))
        s2 = (a * h) ** 2 * torch.cos(ang - phi) ** 2 + (b * h) ** 2 * torch.sin(ang - phi) ** 2
        tau = t - h * (x0 * ca + y0 * sa)
        sino += 2.0 * rho * a * b * h * h * torch.sqrt(torch.clamp(s2 - tau * tau, min=0.0)) / s2
    gen = torch.Generator(device=device).manual_seed(int(seed))
    sino += (0.005 * N) * torch.randn(sino.shape, generator=gen, device=device)
    return sino


def _images(case, seed, device="cuda"):
    """The ellipses sampled at the pixel centres, and 1 % of texture."""
    B, N = case["slices"], case["side"]
    x = (torch.arange(N, device=device, dtype=torch.float32) - 0.5 * (N - 1)) / (0.5 * N)
    X, Y = x.view(1, 1, N), x.view(1, N, 1)
    e = torch.as_tensor(_ellipses(seed, B), device=device, dtype=torch.float32)
    img = torch.zeros((B, N, N), device=device, dtype=torch.float32)
    for i in range(e.shape[1]):
        x0, y0, a, b, phi, rho = (e[:, i, q].view(B, 1, 1) for q in range(6))
        u = (X - x0) * torch.cos(phi) + (Y - y0) * torch.sin(phi)
        v = (Y - y0) * torch.cos(phi) - (X - x0) * torch.sin(phi)
        img += torch.where((u / a) ** 2 + (v / b) ** 2 <= 1.0, rho.expand(B, N, N), torch.zeros((), device=device))
    gen = torch.Generator(device=device).manual_seed(int(seed))
    return img + 0.01 * torch.randn(img.shape, generator=gen, device=device)


def _cone_projections(case, seed, device="cuda"):
    """Chords of random balls seen from the orbit, and 0.5 % of noise."""
    K, Dv, Du, N, Nz, R = (case[k] for k in ("angles", "rows", "bins", "side", "depth", "source"))
    rng = np.random.Generator(np.random.PCG64(seed))
    b = (torch.arange(K, device=device, dtype=torch.float32) * (2.0 * math.pi / K)).view(K, 1, 1)
    s = (torch.arange(Du, device=device, dtype=torch.float32) - 0.5 * (Du - 1)).view(1, 1, Du)
    z = (torch.arange(Dv, device=device, dtype=torch.float32) - 0.5 * (Dv - 1)).view(1, Dv, 1)
    inv = 1.0 / torch.sqrt(R * R + s * s + z * z)
    dx, dy, dz = (-torch.sin(b) * s - R * torch.cos(b)) * inv, (torch.cos(b) * s - R * torch.sin(b)) * inv, z * inv
    out = torch.zeros((K, Dv, Du), device=device, dtype=torch.float32)
    for _ in range(6):
        cx, cy, cz = rng.uniform(-0.3, 0.3, 3) * np.array([N, N, Nz])
        rad, rho = rng.uniform(0.05, 0.15) * min(N, Nz) + 1.0, rng.uniform(-0.5, 1.0)
        wx, wy = float(cx) - R * torch.cos(b), float(cy) - R * torch.sin(b)
        along = wx * dx + wy * dy + float(cz) * dz
        off2 = wx * wx + wy * wy + float(cz) ** 2 - along * along
        out += 2.0 * float(rho) * torch.sqrt(torch.clamp(float(rad) ** 2 - off2, min=0.0))
    gen = torch.Generator(device=device).manual_seed(int(seed))
    return out + (0.005 * N) * torch.randn(out.shape, generator=gen, device=device)


def _batch_inputs(case, seed):
    sinos = []
    for i, (side, K, D) in enumerate(_batch_geometries(case)):
        c = parallel(None, side, K, D, 1)
        sinos.append(_sinograms(c, seed * 1009 + i)[0].contiguous())
    return sinos


def prepare(case, seed):
    op = case["op"]
    if op == "batch":
        geoms, jobs = {}, []
        for (side, K, D), sino in zip(_batch_geometries(case), _batch_inputs(case, seed)):
            if (side, K) not in geoms:
                geoms[side, K] = fbp.Geometry(K, D, side)
            jobs.append((geoms[side, K], sino, torch.empty((side, side), device="cuda")))
        ws = fbp.alloc_workspace(fbp.fbp_batch_workspace_bytes(jobs))
        return dict(op=op, jobs=jobs, ws=ws, images=[j[2] for j in jobs])
    if op == "cone":
        g = _cone_geometry(case)
        return dict(op=op, g=g, proj=_cone_projections(case, seed), vol=torch.empty(g.volume_shape(), device="cuda"),
                    ws=fbp.alloc_workspace(fbp.fbp_cone_workspace_bytes(g)))
    g = _geometry(case)
    if op == "project":
        return dict(op=op, g=g, image=_images(case, seed),
                    sino=torch.empty((case["slices"], case["angles"], case["bins"]), device="cuda"))
    return dict(op=op, g=g, sino=_sinograms(case, seed), precision=case["precision"],
                image=torch.empty((case["slices"], case["side"], case["side"]), device="cuda"),
                ws=fbp.alloc_workspace(fbp.fbp_workspace_bytes(g, case["slices"], case["precision"])))


def run(state):
    op = state["op"]
    if op == "reconstruct":
        return fbp.fbp_reconstruct(state["g"], state["sino"], out=state["image"], workspace=state["ws"],
                                   precision=state["precision"])
    if op == "project":
        return fbp.fbp_project(state["g"], state["image"], out=state["sino"])
    if op == "cone":
        return fbp.fbp_cone_reconstruct(state["g"], state["proj"], out=state["vol"], workspace=state["ws"])
    fbp.fbp_reconstruct_batch(state["jobs"], workspace=state["ws"])
    return state["images"]


# ---------------------------------------------------------------- what a call cannot do without

def _filter_flops(rows, bins):
    """A real FFT convolution of each row: two real transforms of the padded length and a product."""
    L = 2 ** math.ceil(math.log2(max(2, 2 * bins - 1)))
    return rows * (5.0 * L * math.log2(L) + L)


def work(case):
    op = case["op"]
    if op == "batch":
        b = f = 0.0
        for side, K, D in _batch_geometries(case):
            b += 4.0 * (K * D + side * side)
            f += _filter_flops(K, D) + 7.0 * side * side * K
        return {"bytes": b, "flops": f}
    N, K, D = case["side"], case["angles"], case["bins"]
    if op == "cone":
        rows, Nz = K * case["rows"], case["depth"]
        # per voxel and view: the row coordinate, bilinear interpolation, weight and sum
        return {"bytes": 4.0 * (rows * D + N * N * Nz), "flops": _filter_flops(rows, D) + 13.0 * N * N * Nz * K}
    B = case["slices"]
    # per pixel and angle: coordinate, fraction, interpolation and sum; the fan beam's map and weight more
    per = 7.0 if case["source"] == 0 else 16.0
    f = B * per * N * N * K
    if op == "reconstruct":
        f += _filter_flops(B * K, D)
    return {"bytes": 4.0 * B * (K * D + N * N), "flops": f}


# ---------------------------------------------------------------- the same in 64 bits

def _taps(kind, D, dt):
    """dt h(d) for d = -(D-1) .. D-1."""
    d = torch.arange(-D, D + 1, dtype=torch.float64)
    odd = torch.remainder(d, 2) == 1
    ramp = torch.where(odd, -1.0 / (math.pi ** 2 * torch.where(odd, d, torch.ones(())) ** 2 * dt), torch.zeros(()).double())
    ramp[D] = 1.0 / (4.0 * dt)
    if kind == "shepp-logan":
        return (-2.0 / (math.pi ** 2 * dt * (4.0 * d * d - 1.0)))[1:-1]
    if kind == "hann":
        return 0.5 * ramp[1:-1] + 0.25 * (ramp[:-2] + ramp[2:])
    return ramp[1:-1]


def _filtered(sino, kind, dt, half=False, weights=None):
    """Rows [..., D] convolved with the kernel (a Toeplitz product), in 64 bits."""
    D = sino.shape[-1]
    t = _taps(kind, D, dt).to(sino.device) * (0.5 if half else 1.0)
    i = torch.arange(D, device=sino.device)
    T = t[(i.view(1, D) - i.view(D, 1)) + D - 1]          # T[m][n] = tap(n - m)
    x = sino.double()
    if weights is not None:
        x = x * weights
    return (x.reshape(-1, D) @ T).reshape(x.shape)


def _gap_weights(ang):
    a = np.mod(ang, math.pi)
    order = np.argsort(a, kind="stable")
    s = a[order]
    lo, hi = np.concatenate([[s[-1] - math.pi], s[:-1]]), np.concatenate([s[1:], [s[0] + math.pi]])
    w = np.empty_like(a)
    w[order] = 0.5 * (hi - lo)
    return w


def _views(case, device):
    """Per view: bin coordinate [N*N] and weight [N*N] (or a number) of every pixel."""
    N, K, D, R, dt = case["side"], case["angles"], case["bins"], case["source"], case["dt"]
    x = torch.arange(N, device=device, dtype=torch.float64) - 0.5 * (N - 1)
    X, Y = x.view(1, N), x.view(N, 1)
    ang = _angles(case)
    w = _gap_weights(ang) if case["weighting"] == "angle-gaps" else np.full(K, math.pi / K)
    for k in range(K):
        c, s = math.cos(ang[k]), math.sin(ang[k])
        if R > 0:
            L = R - (X * c + Y * s)
            yield R * (Y * c - X * s) / (L * dt) + 0.5 * (D - 1), (2.0 * math.pi / K) * (R / L) ** 2
        else:
            yield (X * c + Y * s) / dt + 0.5 * (D - 1), float(w[k])


def _exact_images(case, q):
    """q [B][K][D] in 64 bits, backprojected."""
    B, K, D = q.shape
    N = case["side"]
    out = torch.zeros((B, N, N), device=q.device, dtype=torch.float64)
    pad = torch.zeros((B, K, D + 4), device=q.device, dtype=torch.float64)
    pad[:, :, 2:-2] = q
    for k, (u, w) in enumerate(_views(case, q.device)):
        u = torch.clamp(u, -1.5, D + 0.5)                 # beyond the ends both neighbours are zero
        i = torch.floor(u)
        f = u - i
        j = (i.long() + 2).reshape(-1)
        row = pad[:, k]
        for b0 in range(0, B, 16):
            r = row[b0:b0 + 16]
            lo, hi = r[:, j].view(-1, N, N), r[:, j + 1].view(-1, N, N)
            out[b0:b0 + 16] += w * (lo + f * (hi - lo))
    return out


def _exact_rows(case, img):
    """img [B][N][N] in 64 bits, forward projected (the adjoint of _exact_images)."""
    B, N, K, D = img.shape[0], case["side"], case["angles"], case["bins"]
    out = torch.zeros((B, K, D + 4), device=img.device, dtype=torch.float64)
    for k, (u, w) in enumerate(_views(case, img.device)):
        u = torch.clamp(u, -1.5, D + 0.5)
        i = torch.floor(u)
        f = u - i
        j = (i.long() + 2).reshape(-1)
        v = (w * img).reshape(B, -1)
        fr = f.reshape(1, -1)
        out[:, k].index_add_(1, j, v * (1.0 - fr))
        out[:, k].index_add_(1, j + 1, v * fr)
    return out[:, :, 2:-2].contiguous()


def _exact_volume(case, q):
    K, Dv, Du, N, Nz, R = (case[k] for k in ("angles", "rows", "bins", "side", "depth", "source"))
    dev = q.device
    x = torch.arange(N, device=dev, dtype=torch.float64) - 0.5 * (N - 1)
    X, Y = x.view(1, N), x.view(N, 1)
    z = (torch.arange(Nz, device=dev, dtype=torch.float64) - 0.5 * (Nz - 1)).view(Nz, 1)
    vol = torch.zeros((Nz, N * N), device=dev, dtype=torch.float64)
    pad = torch.zeros((Dv + 4, Du + 4), device=dev, dtype=torch.float64)
    for k in range(K):
        b = 2.0 * math.pi * k / K
        c, s = math.cos(b), math.sin(b)
        L = R - (X * c + Y * s)
        u = torch.clamp((R * (Y * c - X * s) / L + 0.5 * (Du - 1)).reshape(1, -1), -1.5, Du + 0.5)
        v = torch.clamp(z * (R / L).reshape(1, -1) + 0.5 * (Dv - 1), -1.5, Dv + 0.5)
        pad[2:-2, 2:-2] = q[k]
        iu, iv = torch.floor(u), torch.floor(v)
        fu, fv = u - iu, v - iv
        at = (iv.long() + 2) * (Du + 4) + (iu.long() + 2)
        p = pad.view(-1)
        p0 = p[at] * (1.0 - fu) + p[at + 1] * fu
        at += Du + 4
        p1 = p[at] * (1.0 - fu) + p[at + 1] * fu
        vol += (2.0 * math.pi / K) * ((R / L) ** 2).reshape(1, -1) * (p0 + fv * (p1 - p0))
    return vol.view(Nz, N, N)


def exact(case, seed):
    op = case["op"]
    if op == "batch":
        out = []
        for (side, K, D), sino in zip(_batch_geometries(case), _batch_inputs(case, seed)):
            c = parallel(None, side, K, D, 1)
            out.append(_exact_images(c, _filtered(sino[None], "ramlak", 1.0))[0])
        return out
    if op == "cone":
        proj = _cone_projections(case, seed)
        R, dev = case["source"], proj.device
        s = (torch.arange(case["bins"], device=dev, dtype=torch.float64) - 0.5 * (case["bins"] - 1)).view(1, 1, -1)
        z = (torch.arange(case["rows"], device=dev, dtype=torch.float64) - 0.5 * (case["rows"] - 1)).view(1, -1, 1)
        return _exact_volume(case, _filtered(proj, case["filter"], 1.0, True, R / torch.sqrt(R * R + s * s + z * z)))
    if op == "project":
        return _exact_rows(case, _images(case, seed).double())
    sino = _sinograms(case, seed)
    R, weights = case["source"], None
    if R > 0:
        s = (torch.arange(case["bins"], device=sino.device, dtype=torch.float64) - 0.5 * (case["bins"] - 1)) * case["dt"]
        weights = R / torch.sqrt(R * R + s * s)
    return _exact_images(case, _filtered(sino, case["filter"], case["dt"], R > 0, weights))
