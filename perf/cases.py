"""Performance cases of the library: the work a user's program has it do.

Each case is one pass through the public Python entry points on inputs made
on the GPU from a seed.  Sizes are those of the paper's two ensembles (wind:
15 members of 68x68; Red Sea: 20 members of 500x500), of this repository's
benchmark workloads (128x128 Monte Carlo, the 721x1440x50 ensemble, the
8192x8192 map, the batch of uneven fields, the served stream, a 3D volume),
and odd ones between.

listed()            the named cases, with what each stands for
draw(rng)           one more case of the same ranges
prepare(case, seed) inputs, outputs and handles a program holds before the call
run(state)          one pass, and its outputs
work(case)          bytes and operations one pass cannot do without
exact(case, seed)   run()'s outputs evaluated by plain torch in float64
"""

from __future__ import annotations

import math
import random

import numpy as np
import torch
import torch.nn.functional as F

import paper_2510_01190_amd as P

_DTYPES = {"float32": torch.float32, "float16": torch.float16, "bfloat16": torch.bfloat16}
_MC_POINT_OPS = 60   # Philox words, Box-Muller and the draw, per point and sample
_LCP_OPS = 24        # tail and combination, per LCP value
_FIT_OPS = 8         # Welford, per member value


def listed():
    return [
        # the paper's wind data: the smallest real ensemble, fit and mapped at
        # one isovalue; latency and launch count decide
        dict(name="fit_lcp_68x68_m15_k1", kind="fit_lcp", ny=68, nx=68, members=15, n_iso=1,
             dtype="float32"),
        # a global lat-lon ensemble at several isovalues: member streaming,
        # then a map of ordinary size
        dict(name="fit_lcp_721x1440_m50_k8", kind="fit_lcp", ny=721, nx=1440, members=50, n_iso=8,
             dtype="float32"),
        # the paper's Red Sea pipeline: gradient of the speed per member, fit,
        # closed form at one isovalue
        dict(name="grad_lcp_500x500_m20_k1", kind="grad_lcp", ny=500, nx=500, members=20, n_iso=1,
             dtype="float32"),
        # the largest map: 16 isovalues into a kept output whose rows lie on
        # cache lines, maps interleaved by rows
        dict(name="lcp_8192x8192_k16_interleaved", kind="lcp", ny=8192, nx=8192, n_iso=16,
             dtype="float32", layout="interleaved"),
        # a ragged map, 16-bit storage, an isovalue count that is no power of
        # two, outputs as the call allocates them
        dict(name="lcp_2047x3001_k5_bf16_dense", kind="lcp", ny=2047, nx=3001, n_iso=5,
             dtype="bfloat16", layout="dense"),
        # divergence Gaussians kept by the program, then mapped: an ordinary
        # odd size
        dict(name="two_step_1021x1531_k3_f16", kind="two_step", ny=1021, nx=1531, n_iso=3,
             dtype="float16"),
        # Monte Carlo comparison on a small grid, one isovalue, 2000 samples
        dict(name="mc_128x128_k1_s2000", kind="mc", ny=128, nx=128, n_iso=1, samples=2000,
             dtype="float32"),
        # Monte Carlo comparison on the lat-lon grid, 8 isovalues
        dict(name="mc_721x1440_k8_s1000", kind="mc", ny=721, nx=1440, n_iso=8, samples=1000,
             dtype="float32"),
        # many independent fields of uneven size in one replayed launch
        dict(name="batch_48_fields_k4", kind="batch", fields=48, sizes_seed=4, lo=64, hi=2048,
             n_iso=4, dtype="float32", autotune=False),
        # a serving loop's turn: one new field arrives from the host while
        # slider requests on it and on resident fields are answered
        dict(name="served_512_s6", kind="served", side=512, resident=4, sliders=6, n_iso=4,
             dtype="float32"),
        # geometry of the zero contour (the border of sources and sinks) of a
        # divergence field on a large grid
        dict(name="contour_4096x4096", kind="contour", ny=4096, nx=4096, dtype="float32"),
        # a 3D volume from its moments, rows on cache lines
        dict(name="lcp3d_256x512x384_k4", kind="lcp3d", nz=256, ny=512, nx=384, n_iso=4,
             dtype="float32", fused=True, layout="rows"),
    ]


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["fit_lcp", "grad_lcp", "lcp", "lcp", "two_step", "mc", "batch", "served",
                       "contour", "lcp3d"])
    dtype = rng.choice(["float32", "float32", "float16", "bfloat16"])
    if kind in ("fit_lcp", "grad_lcp"):
        m = rng.randint(10, 50)
        ny = _log_int(rng, 48, 1400)
        nx = min(_log_int(rng, 48, 1500), 721 * 1440 * 50 // (ny * m))
        return dict(kind=kind, ny=ny, nx=nx, members=m, n_iso=rng.randint(1, 8), dtype=dtype)
    if kind == "lcp":
        return dict(kind=kind, ny=_log_int(rng, 64, 8192), nx=_log_int(rng, 64, 8192),
                    n_iso=rng.randint(1, 16), dtype=dtype,
                    layout=rng.choice(["dense", "dense", "rows", "interleaved"]))
    if kind == "two_step":
        return dict(kind=kind, ny=_log_int(rng, 64, 4096), nx=_log_int(rng, 64, 4096),
                    n_iso=rng.randint(1, 16), dtype=dtype)
    if kind == "mc":
        s = _log_int(rng, 100, 2000)
        ny = _log_int(rng, 64, 1000)
        nx = min(_log_int(rng, 64, 1500), 721 * 1440 * 1000 // (ny * s))
        return dict(kind=kind, ny=ny, nx=nx, n_iso=rng.randint(1, 8), samples=s, dtype=dtype)
    if kind == "batch":
        return dict(kind=kind, fields=_log_int(rng, 8, 64), sizes_seed=rng.randint(0, 10 ** 6),
                    lo=64, hi=_log_int(rng, 256, 2048), n_iso=rng.randint(1, 8), dtype=dtype,
                    autotune=rng.random() < 0.5)
    if kind == "served":
        return dict(kind=kind, side=_log_int(rng, 256, 1500), resident=rng.randint(2, 6),
                    sliders=rng.randint(3, 10), n_iso=rng.randint(1, 4), dtype=dtype)
    if kind == "contour":
        return dict(kind=kind, ny=_log_int(rng, 64, 4096), nx=_log_int(rng, 64, 4096),
                    dtype="float32")
    nz, ny = _log_int(rng, 24, 256), _log_int(rng, 24, 512)
    nx = min(_log_int(rng, 24, 512), 256 * 512 * 384 // (nz * ny))
    return dict(kind=kind, nz=nz, ny=ny, nx=nx, n_iso=rng.randint(1, 8), dtype=dtype,
                fused=rng.random() < 0.6, layout=rng.choice(["dense", "rows"]))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed: int, salt: int = 0):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7fffffffffff)
    return g


def _smooth(g, ny: int, nx: int, step: float = 14.0, amp: float = 0.8):
    """A smooth random plane: normal values `step` points apart, interpolated."""
    cy, cx = max(4, int(ny / step) + 2), max(4, int(nx / step) + 2)
    c = torch.randn(1, 1, cy, cx, generator=g, device="cuda") * amp
    return F.interpolate(c, size=(ny, nx), mode="bicubic", align_corners=True)[0, 0].contiguous()


def _moments2(g, ny: int, nx: int, dtype, sigma=(0.05, 0.5)):
    """Mean and variance planes of U and V: smooth means, spread drawn per
    point and component."""
    planes = []
    for _ in range(2):
        sd = torch.rand(ny, nx, generator=g, device="cuda") * (sigma[1] - sigma[0]) + sigma[0]
        planes += [_smooth(g, ny, nx), sd * sd]
    return [p.to(dtype) for p in planes]


def _ensemble(g, ny: int, nx: int, m: int, dtype):
    """Members of U and V: a smooth base plus noise of smoothly varying spread."""
    out = []
    for _ in range(2):
        base = _smooth(g, ny, nx, step=40.0, amp=2.0)
        sd = 0.1 + 1.4 * torch.sigmoid(_smooth(g, ny, nx, step=150.0, amp=1.5))
        x = torch.randn(m, ny, nx, generator=g, device="cuda")
        out.append(x.mul_(sd).add_(base).to(dtype))
    return out


def _moments3(g, nz: int, ny: int, nx: int, dtype):
    """Six moment volumes: means are sums of separable waves (1-4 periods an
    axis), spread drawn per point and component."""
    planes = []
    n = (nx, ny, nz)
    for own in range(3):
        mean = torch.zeros(nz, ny, nx, device="cuda")
        for _ in range(4):
            r = torch.rand(7, generator=g, device="cuda").tolist()
            k = [1.0 + 3.0 * r[a] for a in range(3)]
            amp = (2.0 * r[6] - 1.0) * n[own] / (2.0 * math.pi * k[own])
            fx, fy, fz = (torch.sin(torch.arange(n[a], device="cuda") * (2.0 * math.pi * k[a] / n[a])
                                    + 2.0 * math.pi * r[3 + a]) for a in range(3))
            mean += (amp * fz)[:, None, None] * (fy[:, None] * fx[None, :])[None]
        sd = torch.rand(nz, ny, nx, generator=g, device="cuda") * 0.45 + 0.05
        planes += [mean.to(dtype), (sd * sd).to(dtype)]
    return planes


def _dd(f, axis: int):
    return torch.gradient(f, dim=axis)[0]


def _isovalues(div, k: int):
    """k values at quantiles of a divergence, as the program's float32 array."""
    v = div.reshape(-1)
    v = v[:: max(1, v.numel() // 200_000)].double()
    q = torch.linspace(0.1, 0.9, k, dtype=torch.float64, device=v.device) if k > 1 else \
        torch.tensor([0.5], dtype=torch.float64, device=v.device)
    return torch.quantile(v, q).cpu().numpy().astype(np.float32)


def _sizes(case):
    r = random.Random(case["sizes_seed"])
    return [(_log_int(r, case["lo"], case["hi"]), _log_int(r, case["lo"], case["hi"]))
            for _ in range(case["fields"])]


def _speed_gradient(u, v):
    s = torch.sqrt(u * u + v * v)
    return _dd(s, -1), _dd(s, -2)


def _inputs(case, seed):
    """The case's inputs: device tensors (host planes for the served fields)
    and isovalues."""
    g = _gen(seed)
    kind, dt = case["kind"], _DTYPES[case["dtype"]]
    if kind in ("fit_lcp", "grad_lcp"):
        u, v = _ensemble(g, case["ny"], case["nx"], case["members"], dt)
        a, b = u.float(), v.float()
        if kind == "grad_lcp":
            a, b = _speed_gradient(a, b)
        div = _dd(a.mean(0), 1) + _dd(b.mean(0), 0)
        return dict(u=u, v=v, iso=_isovalues(div, case["n_iso"]))
    if kind in ("lcp", "two_step", "mc"):
        m = _moments2(g, case["ny"], case["nx"], dt)
        div = _dd(m[0].float(), 1) + _dd(m[2].float(), 0)
        return dict(m=m, iso=_isovalues(div, case["n_iso"]))
    if kind == "batch":
        fields = []
        for ny, nx in _sizes(case):
            m = _moments2(g, ny, nx, dt)
            fields.append((m, _isovalues(_dd(m[0].float(), 1) + _dd(m[2].float(), 0),
                                         case["n_iso"])))
        return dict(fields=fields)
    if kind == "served":
        n = case["side"]
        host, isos = [], []
        for _ in range(case["resident"] + 1):
            m = _moments2(g, n, n, dt)
            isos.append(_isovalues(_dd(m[0].float(), 1) + _dd(m[2].float(), 0), case["n_iso"]))
            host.append([p.cpu() for p in m])
        return dict(host=host, isos=isos)
    if kind == "contour":
        # the sizes alone decide which points lie above zero (so the number of
        # segments is the case's own), the seed every value
        ny, nx = case["ny"], case["nx"]
        shape = _gen(ny * 8209 + nx, 1)
        f = _dd(_smooth(shape, ny, nx), 1) + _dd(_smooth(shape, ny, nx), 0)
        f *= 0.25 + torch.sigmoid(_smooth(g, ny, nx, step=6.0, amp=1.5))
        return dict(field=f.contiguous(), iso=0.0)
    m = _moments3(g, case["nz"], case["ny"], case["nx"], dt)
    div = _dd(m[0].float(), 2) + _dd(m[2].float(), 1) + _dd(m[4].float(), 0)
    return dict(m=m, iso=_isovalues(div, case["n_iso"]))


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    s["kind"] = kind
    if kind == "lcp" and case["layout"] != "dense":
        s["out"] = P.empty_lcp(case["n_iso"], case["ny"], case["nx"],
                               interleave_rows=case["layout"] == "interleaved")
    elif kind == "mc":
        s.update(samples=case["samples"], seed=int(seed) & 0x7fffffff)
    elif kind == "batch":
        s["batch"] = P.Batch([dict(mean_u=m[0], var_u=m[1], mean_v=m[2], var_v=m[3],
                                   isovalues=torch.from_numpy(iso).cuda())
                              for m, iso in s["fields"]], autotune=case["autotune"])
        s["outs"] = [f["lcp"] for f in s["batch"].fields]
    elif kind == "served":
        n, k = case["side"], case["n_iso"]
        size = 4 if case["dtype"] == "float32" else 2
        # room for the resident fields and two new ones being uploaded
        budget = n * n * (8 * (case["resident"] + 3) + 3 * 4 * size) + (8 << 20)
        srv = P.Server(budget, n_streams=2)
        srv.wait(srv.put_field(0, *s["host"][0]))
        for f in range(1, case["resident"]):
            srv.wait(srv.put_field(f, *s["host"][f]))
        s.update(server=srv, next_id=1000, resident=case["resident"],
                 outs=[torch.empty(k, n - 1, n - 1, device="cuda") for _ in range(case["sliders"])])
    elif kind == "lcp3d":
        s["fused"] = case["fused"]
        if case["layout"] == "rows":
            s["out"] = P.empty_lcp_3d(case["n_iso"], case["nz"], case["ny"], case["nx"])
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "fit_lcp":
        mom = P.moments(s["u"], s["v"])
        return [*mom, P.lcp_from_moments(*mom, s["iso"])]
    if kind == "grad_lcp":
        mom = P.speed_gradient_moments(s["u"], s["v"])
        return [*mom, P.lcp_from_moments(*mom, s["iso"])]
    if kind == "lcp":
        return P.lcp_from_moments(*s["m"], s["iso"], out=s.get("out"))
    if kind == "two_step":
        dm, dv = P.divergence_gaussian(*s["m"])
        return [dm, dv, P.lcp(dm, dv, s["iso"])]
    if kind == "mc":
        return P.mc_lcp(*s["m"], s["iso"], s["samples"], s["seed"])
    if kind == "batch":
        s["batch"].launch()
        return s["outs"]
    if kind == "served":
        srv, n = s["server"], s["resident"]
        fid = s["next_id"]
        s["next_id"] += 1
        tickets = [srv.put_field(fid, *s["host"][n])]
        for q, out in enumerate(s["outs"]):  # every (n+1)-th request is on the new field
            f = q % (n + 1)
            tickets.append(srv.submit_lcp(fid if f == n else f, s["isos"][f], out))
        for t in tickets:
            if srv.wait(t) != 0:
                raise RuntimeError("a served request failed")
        return s["outs"]
    if kind == "contour":
        return P.isocontour(s["field"], s["iso"])
    if s["fused"]:
        return P.lcp_3d_from_moments(*s["m"], s["iso"], out=s.get("out"))
    dm, dv = P.divergence_gaussian_3d(*s["m"])
    return [dm, dv, P.lcp_3d(dm, dv, s["iso"], out=s.get("out"))]


# ---------------------------------------------------------------------------
# What one pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    b = 4 if case["dtype"] == "float32" else 2
    if kind == "batch":
        pts = sum(ny * nx for ny, nx in _sizes(case))
        vals = sum((ny - 1) * (nx - 1) for ny, nx in _sizes(case)) * case["n_iso"]
        return dict(bytes=4 * b * pts + 4 * vals, flops=_LCP_OPS * vals)
    if kind == "served":
        n = case["side"]
        vals = case["sliders"] * case["n_iso"] * (n - 1) ** 2
        return dict(bytes=4 * b * n * n + 4 * vals, flops=_LCP_OPS * vals)
    pts = case.get("nz", 1) * case["ny"] * case["nx"]
    cells = max(1, case.get("nz", 2) - 1) * (case["ny"] - 1) * (case["nx"] - 1)
    k = case.get("n_iso", 1)
    if kind in ("fit_lcp", "grad_lcp"):
        return dict(bytes=2 * case["members"] * b * pts + 16 * pts + 4 * k * cells,
                    flops=2 * _FIT_OPS * case["members"] * pts + _LCP_OPS * k * cells)
    if kind == "lcp":
        return dict(bytes=4 * b * pts + 4 * k * cells, flops=_LCP_OPS * k * cells)
    if kind == "two_step":
        return dict(bytes=4 * b * pts + 8 * pts + 4 * k * cells, flops=_LCP_OPS * k * cells)
    if kind == "mc":
        return dict(bytes=4 * b * pts + 4 * k * cells,
                    flops=case["samples"] * (_MC_POINT_OPS * pts + 6.0 * cells))
    if kind == "contour":
        return dict(bytes=4 * pts, flops=4.0 * cells)
    extra = 0 if case["fused"] else 8 * pts
    return dict(bytes=6 * b * pts + extra + 4 * k * cells, flops=2 * _LCP_OPS * k * cells)


# ---------------------------------------------------------------------------
# The same outputs in float64
# ---------------------------------------------------------------------------

def _var_dd(v, axis: int):
    """Variance of the difference quotient along an axis (spacing 1)."""
    n = v.shape[axis]
    lo = torch.arange(n, device=v.device).sub(1).clamp_(min=0)
    hi = torch.arange(n, device=v.device).add(1).clamp_(max=n - 1)
    w = torch.full((n,), 0.25, dtype=v.dtype, device=v.device)
    w[0] = w[-1] = 1.0
    shape = [1] * v.dim()
    shape[axis] = n
    return (v.index_select(axis, lo) + v.index_select(axis, hi)) * w.reshape(shape)


def _lcp64(mu, var, iso):
    """1 - prod P(above) - prod P(below) over each cell's corners, float64."""
    rs = torch.rsqrt(var * 2.0)
    out = torch.empty((len(iso),) + tuple(n - 1 for n in mu.shape), dtype=torch.float64,
                      device=mu.device)
    for q, c in enumerate(iso):
        z = (mu - float(c)) * rs
        total = None
        for p in (0.5 * torch.erfc(-z), 0.5 * torch.erfc(z)):
            for axis in range(p.dim()):
                n = p.shape[axis]
                p = p.narrow(axis, 0, n - 1) * p.narrow(axis, 1, n - 1)
            total = p if total is None else total + p
        out[q] = 1.0 - total
    return out


def _div64(m):
    """Eq. 2-3 in float64 from the stored planes (2D: U, V; 3D: U, V, W)."""
    mu = var = None
    for c in range(len(m) // 2):
        axis = m[0].dim() - 1 - c
        a, b = _dd(m[2 * c].double(), axis), _var_dd(m[2 * c + 1].double(), axis)
        mu, var = (a, b) if mu is None else (mu + a, var + b)
    return mu, var


def _fit64(x):
    mean = x.mean(0)
    var = torch.zeros_like(mean)
    for xm in x:
        var += (xm - mean) ** 2
    return mean, var / (x.shape[0] - 1)


def _philox(point, pair: int, seed: int):
    mask = 0xffffffff
    k0, k1 = seed & mask, (seed >> 32) & mask
    x, y = point, torch.full_like(point, pair)
    z, w = torch.zeros_like(point), torch.zeros_like(point)
    for _ in range(10):
        p0, p1 = x * 0xD2511F53, z * 0xCD9E8D57  # the low 64 bits are what is used
        x, y, z, w = (((p1 >> 32) & mask) ^ y ^ k0, p1 & mask,
                      ((p0 >> 32) & mask) ^ w ^ k1, p0 & mask)
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return x, y, z, w


def _mc64(m, iso, samples: int, seed: int):
    mu, mv = m[0].double(), m[2].double()
    su, sv = m[1].double().sqrt(), m[3].double().sqrt()
    point = torch.arange(mu.numel(), dtype=torch.int64, device=mu.device)
    c = torch.from_numpy(iso.astype(np.float64)).to(mu.device)[:, None, None]
    count = torch.zeros((len(iso), mu.shape[0] - 1, mu.shape[1] - 1), dtype=torch.int32,
                        device=mu.device)
    for pair in range((samples + 1) // 2):
        w = _philox(point, pair, seed)
        for s in range(2):
            if 2 * pair + s >= samples:
                continue
            r = torch.sqrt(-2.0 * torch.log((w[2 * s].double() + 1.0) * 2.0 ** -32))
            a = w[2 * s + 1].double() * (2.0 * math.pi * 2.0 ** -32)
            u = mu + su * (r * torch.cos(a)).reshape(mu.shape)
            v = mv + sv * (r * torch.sin(a)).reshape(mu.shape)
            d = _dd(u, 1) + _dd(v, 0)
            lo, hi = torch.minimum(d[1:], d[:-1]), torch.maximum(d[1:], d[:-1])
            lo = torch.minimum(lo[:, 1:], lo[:, :-1])
            hi = torch.maximum(hi[:, 1:], hi[:, :-1])
            count += (lo[None] < c) & (hi[None] >= c)
    return count.double() / samples


# edges a and b of each case's segment (0 bottom, 1 right, 2 top, 3 left); the
# saddles 5 and 10 are decided by the cell centre
_EDGE_A = [0, 3, 0, 3, 1, 0, 0, 2, 2, 0, 0, 1, 3, 0, 3, 0]
_EDGE_B = [0, 0, 1, 1, 2, 0, 2, 3, 3, 2, 0, 2, 1, 1, 0, 0]


def _contour64(f, c: float):
    f = f.double()
    v00, v10, v11, v01 = f[:-1, :-1], f[:-1, 1:], f[1:, 1:], f[1:, :-1]
    case = (v00 >= c).int() + 2 * (v10 >= c).int() + 4 * (v11 >= c).int() + 8 * (v01 >= c).int()
    saddle = (case == 5) | (case == 10)
    some = (case != 0) & (case != 15)
    at = torch.nonzero(torch.stack([some, saddle], -1))  # row-major: cell, then its segment
    j, i, second = at[:, 0], at[:, 1], at[:, 2] == 1
    p00, p10, p11, p01 = (v[j, i] for v in (v00, v10, v11, v01))
    cs, sad = case[j, i].long(), saddle[j, i]
    ea = torch.tensor(_EDGE_A, device=f.device)[cs]
    eb = torch.tensor(_EDGE_B, device=f.device)[cs]
    join = (cs == 5) == (((p00 + p10) + (p11 + p01)) * 0.25 >= c)
    sel = torch.where
    ea = sel(sad, sel(second, sel(join, 2, 1), sel(join, 0, 3)), ea)
    eb = sel(sad, sel(second, sel(join, 3, 2), sel(join, 1, 0)), eb)

    def point(e):
        p = sel(e == 1, p10, sel(e == 2, p01, p00))
        q = sel(e == 0, p10, sel(e == 3, p01, p11))
        t = (c - p) / (q - p)
        along_x = (e == 0) | (e == 2)
        return (i + (e == 1).long()).double() + sel(along_x, t, 0.0), \
            (j + (e == 2).long()).double() + sel(along_x, 0.0, t)

    return torch.stack([*point(ea), *point(eb)], -1)


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("fit_lcp", "grad_lcp"):
        u, v = s["u"].double(), s["v"].double()
        if kind == "grad_lcp":
            u, v = _speed_gradient(u, v)
        m = [*_fit64(u), *_fit64(v)]
        return [*m, _lcp64(*_div64(m), s["iso"])]
    if kind == "lcp":
        return _lcp64(*_div64(s["m"]), s["iso"])
    if kind == "two_step":
        dm, dv = _div64(s["m"])
        return [dm, dv, _lcp64(dm, dv, s["iso"])]
    if kind == "mc":
        return _mc64(s["m"], s["iso"], case["samples"], int(seed) & 0x7fffffff)
    if kind == "batch":
        return [_lcp64(*_div64(m), iso) for m, iso in s["fields"]]
    if kind == "served":
        n, maps = case["resident"], []
        for q in range(case["sliders"]):
            f = q % (n + 1)
            maps.append(_lcp64(*_div64([p.cuda() for p in s["host"][f]]), s["isos"][f]))
        return maps
    if kind == "contour":
        return _contour64(s["field"], s["iso"])
    dm, dv = _div64(s["m"])
    maps = _lcp64(dm, dv, s["iso"])
    return maps if case["fused"] else [dm, dv, maps]
