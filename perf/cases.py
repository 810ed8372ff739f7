"""The work that programs have this library do, as timed and compared cases.

A case is one call (or one step of a loop) through the public entry points:
single builds from a small molecule to a capsid-like shell, builds into the
caller's own tensors, builds from and to host arrays, a batch of molecules,
recorded builds replayed on the frames of a trajectory, one complex per alpha
value of a sweep, and the union's volume and area with their gradients.

Inputs are synthetic molecules: atoms at 0.05 per cubic angstrom whose centres
keep about 2.4 A apart, in a ball or in a shell of inner radius 0.7 R_out, with
the radii of C, N, O and S (p .62 .17 .19 .02), or solvent-accessible radii
(1.4 A more), in random input order. Centres come from a periodic block of
relaxed points, jittered. A case fixes its molecules up to how they lie in
space and in which order their atoms come (so that every seed has as many
simplices); the seed turns, mirrors and shifts each molecule and shuffles its
atoms.
"""
import math

import numpy as np
import torch

import paper_1908_05944_amd as acx

DENSITY = 0.05
TILE = 2048  # atoms of the periodic block
TILE_SIDE = (TILE / DENSITY) ** (1.0 / 3.0)
JITTER = 0.05


def listed():
    return [
        # the smallest molecule of a structure database: a call is launches and waits
        {"name": "build_260", "call": "build", "n": 260, "alpha": 0.0, "radii": "vdw"},
        # a small protein inside a tight loop that owns its output tensors
        {"name": "noalloc_1003_a1", "call": "noalloc", "n": 1003, "alpha": 1.0, "radii": "vdw"},
        # a medium protein at a larger alpha (cavities, shape filtrations)
        {"name": "build_16647_a2", "call": "build", "n": 16647, "alpha": 2.0, "radii": "vdw"},
        # an ordinary large assembly
        {"name": "build_100k", "call": "build", "n": 100000, "alpha": 0.0, "radii": "vdw"},
        # the same with solvent-accessible radii: long neighbour rows
        {"name": "build_100k_sas", "call": "build", "n": 100000, "alpha": 0.0, "radii": "sas"},
        # a capsid-like shell, the largest single build
        {"name": "build_3m_shell", "call": "build", "n": 3000000, "alpha": 0.0, "radii": "vdw", "shape": "shell",
         "cell_mA": 3600},
        # a library of molecules of very different sizes in one call
        {"name": "batch_512", "call": "batch", "mols": 512, "lo": 500, "hi": 50000, "alpha": 0.0, "radii": "vdw"},
        # the frames of a trajectory through a recorded build: new coordinates, replay, result
        {"name": "plan_58674", "call": "plan", "n": 58674, "alpha": 0.0, "radii": "vdw"},
        # one step of an optimisation over volume and area: build, forward, backward
        {"name": "step_100k", "call": "step", "n": 100000, "alpha": 0.0, "radii": "vdw"},
        # volume, area and gradient again and again on a complex held fixed
        {"name": "measure_4001", "call": "measure", "n": 4001, "alpha": 0.0, "radii": "vdw"},
        # a filtration: the complexes of several alpha values of one molecule
        {"name": "sweep_100k", "call": "sweep", "n": 100000, "alpha": 2.0, "alphas": 5, "radii": "vdw"},
        # a program without device memory of its own: arrays in, arrays out
        {"name": "host_58674_a1", "call": "host", "n": 58674, "alpha": 1.0, "radii": "vdw"},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    call = rng.choice(["build", "build", "build", "noalloc", "batch", "plan", "step", "measure", "sweep", "host"])
    case = {"call": call, "alpha": 0.0, "radii": "vdw"}
    if call == "build":
        case["n"] = size(260, 1000000)
        case["alpha"] = rng.choice([0.0, 0.0, 0.5, 1.0, 2.0])
        if case["n"] <= 200000 and rng.random() < 0.25:
            case.update(alpha=0.0, radii="sas")
        if case["n"] > 20000 and rng.random() < 0.3:
            case["shape"] = "shell"
    elif call == "noalloc":
        case["n"] = size(260, 20000)
        case["alpha"] = rng.choice([0.0, 1.0])
    elif call == "batch":
        case["mols"] = size(4, 256)
        case["lo"], case["hi"] = 500, size(2000, 50000)
    elif call == "plan":
        case["n"] = size(260, 200000)
    elif call in ("step", "measure"):
        case["n"] = size(260, 200000)
        if case["n"] <= 50000 and rng.random() < 0.2:
            case["radii"] = "sas"
    elif call == "sweep":
        case["n"] = size(1000, 200000)
        case["alpha"] = rng.choice([0.5, 1.0, 2.0])
        case["alphas"] = rng.randint(2, 7)
    else:
        case["n"] = size(260, 100000)
        case["alpha"] = rng.choice([0.0, 1.0])
    return case


# --------------------------------------------------------------------------
# Inputs


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


_tiles = {}


def _tile():
    """TILE points in a periodic cube, about 2.4 A apart: random points pushed apart."""
    dev = _device()
    if dev not in _tiles:
        p = torch.from_numpy(np.random.RandomState(11).rand(TILE, 3) * TILE_SIDE).to(dev)
        eye = torch.eye(TILE, dtype=torch.bool, device=dev)
        for _ in range(150):
            d = p[:, None, :] - p[None, :, :]
            d = d - TILE_SIDE * torch.round(d / TILE_SIDE)
            r = d.square().sum(-1).sqrt().masked_fill(eye, 1e9)
            push = (2.42 - r).clamp(min=0.0) / (2.0 * r)
            p = torch.remainder(p + (push[..., None] * d).sum(1), TILE_SIDE)
        _tiles[dev] = p
    return _tiles[dev]


def _molecule(n, salt, shape, radii):
    """n atoms around the origin (n x 3 in milli-angstrom, and n radii in angstrom) that the case fixes."""
    dev = _device()
    rng = np.random.RandomState((n + 7919 * salt) % (1 << 31))
    inner = 0.7 if shape == "shell" else 0.0
    r_out = (3.0 * n / (4.0 * math.pi * DENSITY * (1.0 - inner ** 3))) ** (1.0 / 3.0)
    shift = torch.from_numpy(rng.rand(3) * TILE_SIDE).to(dev)
    reach = r_out * 1.03 + 3.0
    k = int(math.ceil(reach / TILE_SIDE)) + 1
    c = torch.arange(-k, k, device=dev, dtype=torch.float64) * TILE_SIDE
    corner = torch.stack(torch.meshgrid(c, c, c, indexing="ij"), -1).reshape(-1, 3) + shift
    dist = (corner + TILE_SIDE / 2).square().sum(1).sqrt()
    half = TILE_SIDE * math.sqrt(3.0) / 2
    corner = corner[(dist < reach + half) & (dist > inner * r_out - half)]
    p = (corner[:, None, :] + _tile()[None, :, :]).reshape(-1, 3)
    r2 = p.square().sum(1)
    if inner:
        p = p[r2 >= (inner * r_out) ** 2]
        r2 = p.square().sum(1)
    p = p[torch.argsort(r2, stable=True)[:n]]
    g = torch.Generator(device=dev).manual_seed(int(rng.randint(1 << 30)))
    p = torch.round((p + JITTER * torch.randn(n, 3, generator=g, device=dev, dtype=torch.float64)) * 1000.0)
    u = torch.rand(n, generator=g, device=dev, dtype=torch.float64)
    rad = torch.where(u < 0.62, 1.70, torch.where(u < 0.79, 1.55, torch.where(u < 0.98, 1.52, 1.80))).double()
    return p, rad + (1.4 if radii == "sas" else 0.0)


def _placed(mol, rng):
    """The molecule turned, mirrored and shifted, its atoms shuffled (angstrom)."""
    p, r = mol
    axes = torch.from_numpy(rng.permutation(3)).to(p.device)
    sign = torch.from_numpy(rng.choice([-1.0, 1.0], 3)).to(p.device)
    shift = torch.from_numpy(rng.randint(-100000, 100001, 3).astype(np.float64)).to(p.device)
    g = torch.Generator(device=p.device).manual_seed(int(rng.randint(1 << 30)))
    order = torch.randperm(len(r), generator=g, device=p.device)
    return ((p[:, axes] * sign + shift)[order] / 1000.0).contiguous(), r[order].contiguous()


def _alphas(case):
    return [case["alpha"] * k / (case["alphas"] - 1) for k in range(case["alphas"])]


def _options(case):
    return {"cell_mA": case["cell_mA"]} if case.get("cell_mA") else None


def _sizes(case):
    """Sizes of a batch's molecules: log-uniform."""
    rng = np.random.RandomState((999 + 7 * case["mols"] + case["hi"]) % (1 << 31))
    u = rng.rand(case["mols"])
    return np.rint(np.exp(math.log(case["lo"]) + u * math.log(case["hi"] / case["lo"]))).astype(np.int64)


def _inputs(case, seed):
    rng = np.random.RandomState(seed % (1 << 31))
    if case["call"] == "batch":
        sizes = _sizes(case)
        mols = [_placed(_molecule(int(n), m, "ball", case["radii"]), rng) for m, n in enumerate(sizes)]
        off = np.concatenate([[0], np.cumsum(sizes)])
        return torch.cat([m[0] for m in mols]), torch.cat([m[1] for m in mols]), off
    x, r = _placed(_molecule(case["n"], 0, case.get("shape", "ball"), case["radii"]), rng)
    return x, r, np.array([0, case["n"]], dtype=np.int64)


def prepare(case, seed):
    x, r, off = _inputs(case, seed)
    s = {"case": case, "x": x, "r": r, "off": off, "options": _options(case)}
    call = case["call"]
    if call == "host":
        s["x"], s["r"] = x.cpu().numpy(), r.cpu().numpy()
    elif call == "noalloc":
        cap = [case["n"] * k for k in (1, 8, 10, 4)]
        s["simp"] = [torch.empty(cap[d], d + 1, dtype=torch.int32, device=x.device) for d in range(4)]
        s["size"] = [torch.empty(cap[d], dtype=torch.float64, device=x.device) for d in range(4)]
    elif call == "plan":
        # the tensor the plan records (another frame of the trajectory first),
        # and the frame that a pass writes into it
        s["frame"] = x.clone()
        g = torch.Generator(device=x.device).manual_seed(seed % (1 << 31))
        x += torch.round(JITTER * 1000.0 * torch.randn(x.shape, generator=g, device=x.device, dtype=x.dtype)) / 1000.0
        s["plan"] = acx.Plan(x, r, off, case["alpha"])
    elif call in ("measure", "step"):
        s["grad"] = torch.tensor([1.0, 0.5], dtype=torch.float64, device=x.device)
        if call == "measure":
            s["complex"] = acx.ac_alpha_complex_device(x, r, case["alpha"])
    return s


# --------------------------------------------------------------------------
# One pass


class _Rows:
    """Device rows of a result as a tensor source (keeps the result alive)."""

    def __init__(self, c, ptr, shape, typestr):
        self._complex = c
        self.__cuda_array_interface__ = {"shape": shape, "typestr": typestr, "data": (ptr, False), "version": 2}


def _tensors(c):
    """[simplices, sizes] of dimensions 0..3 as device tensors over the result's own arrays."""
    out = []
    for d in range(4):
        m = c.count(d)
        if m == 0:
            out += [torch.empty(0, d + 1, dtype=torch.int32, device="cuda"),
                    torch.empty(0, dtype=torch.float64, device="cuda")]
            continue
        ps, pz = c.device_pointers(d)
        out += [torch.as_tensor(_Rows(c, ps, (m, d + 1), "<i4"), device="cuda"),
                torch.as_tensor(_Rows(c, pz, (m,), "<f8"), device="cuda")]
    return out


def run(s):
    case = s["case"]
    call, alpha = case["call"], case["alpha"]
    if call == "build":
        return _tensors(acx.ac_alpha_complex_device(s["x"], s["r"], alpha, options=s["options"]))
    if call == "noalloc":
        m = acx.ac_alpha_complex_noalloc(s["x"], s["r"], alpha, s["simp"], s["size"])
        return [t for d in range(4) for t in (s["simp"][d][:m[d]], s["size"][d][:m[d]])]
    if call == "batch":
        return _tensors(acx.ac_alpha_complex_batch(s["x"], s["r"], s["off"], alpha))
    if call == "plan":
        s["x"].copy_(s["frame"])
        s["plan"].launch()
        return _tensors(s["plan"].result())
    if call == "step":
        x = s["x"].detach().requires_grad_(True)
        r = s["r"].detach().requires_grad_(True)
        c = acx.ac_alpha_complex_device(s["x"], s["r"], alpha)
        va = acx.UnionMeasure.apply(x, r, c)
        va.backward(s["grad"])
        return [va.detach(), x.grad, r.grad]
    if call == "measure":
        return list(acx.ac_union_measure_fused(s["complex"], s["x"], s["r"], s["grad"]))
    if call == "sweep":
        return [_tensors(c) for c in acx.ac_alpha_sweep_device(s["x"], s["r"], _alphas(case))]
    c = acx.ac_alpha_complex(s["x"], s["r"], alpha)
    return [t for d in range(4) for t in (c.simplices(d), c.sizes(d))]


# simplices of K_alpha per ball, dimensions 0..3, of such molecules
_PER_BALL = {0.0: (1.0, 3.5, 2.1, 0.18), 0.5: (1.0, 4.3, 3.6, 0.7), 1.0: (1.0, 5.2, 5.8, 1.7),
             2.0: (1.0, 6.3, 8.9, 3.6), "sas": (1.0, 7.1, 12.1, 6.0)}



def _output_bytes(n, alpha, radii):
    near = min((0.0, 0.5, 1.0, 2.0), key=lambda a: abs(a - alpha))
    per = _PER_BALL["sas" if radii == "sas" else near]
    return n * sum(m * (4 * (d + 1) + 8) for d, m in enumerate(per))


def work(case):
    """Inputs (32 bytes a ball) read once, outputs written once; float64
    operations: orthosizes and emptiness tests of the candidates, or the
    corner terms of the union measure."""
    call, radii = case["call"], case["radii"]
    n = int(_sizes(case).sum()) if call == "batch" else case["n"]
    flops_per_ball = 8000.0 if radii == "sas" else 1300.0 * (1.0 + 2.0 * case["alpha"])
    corners = n * (75.0 if radii == "sas" else 15.0)  # (simplex, corner) pairs
    if call == "measure":
        return {"bytes": n * 64.0 + 4.0 * corners, "flops": corners * 400.0}
    if call == "step":
        return {"bytes": n * 64.0, "flops": n * flops_per_ball + corners * 600.0}
    if call == "sweep":
        out = sum(_output_bytes(n, a, radii) for a in _alphas(case))
        return {"bytes": n * 32.0 + out, "flops": n * flops_per_ball}
    return {"bytes": n * 32.0 + _output_bytes(n, case["alpha"], radii), "flops": n * flops_per_ball}


# --------------------------------------------------------------------------
# The same in 64 bits, from the definition


def _pairs(start, count):
    """(row, index) of every index in [start, start + count) of each row."""
    row = torch.repeat_interleave(torch.arange(len(count), device=count.device), count)
    first = torch.cumsum(count, 0) - count
    return row, torch.arange(len(row), device=count.device) - first[row] + start[row]


def _neighbours(X, W, aq):
    """Rows (i sorted) and columns of every ordered pair whose grown balls meet."""
    n = len(W)
    reach = 2.0 * math.sqrt(max(float(W.max()) + aq, 0.0))
    side = max(int(math.ceil(reach)), 1)
    c = torch.div(X - X.min(0).values, side, rounding_mode="floor") + 1
    ny, nz = int(c[:, 1].max()) + 2, int(c[:, 2].max()) + 2
    key = (c[:, 0] * ny + c[:, 1]) * nz + c[:, 2]
    order = torch.argsort(key)
    sk = key[order]
    rows, cols = [], []
    for dx in (-1, 0, 1):
        for dy in (-1, 0, 1):
            k = key + (dx * ny + dy) * nz
            lo, hi = torch.searchsorted(sk, k - 1), torch.searchsorted(sk, k + 1, right=True)
            i, at = _pairs(lo, hi - lo)
            j = order[at]
            d2 = (X[i] - X[j]).square().sum(1)
            a, b = W[i] + aq, W[j] + aq
            L = d2 - a - b
            meet = (i != j) & (a >= 0) & (b >= 0) & ((L <= 0) | (L * L <= 4 * a * b))
            rows.append(i[meet])
            cols.append(j[meet])
    i, j = torch.cat(rows), torch.cat(cols)
    o = torch.argsort(i * n + j)
    return i[o], j[o]


def _centres(X, W, S):
    """Ortho-centre relative to the first vertex and OrthoSize of each row of S."""
    p = X[S].double()
    w = W[S].double()
    if S.shape[1] == 1:
        return torch.zeros(len(S), 3, dtype=torch.float64, device=X.device), -w[:, 0]
    a = p[:, 1:] - p[:, :1]
    beta = a.square().sum(-1) - w[:, 1:] + w[:, :1]
    if S.shape[1] == 2:
        c = a[:, 0] * (beta[:, :1] / (2.0 * a[:, 0].square().sum(-1, keepdim=True)))
    elif S.shape[1] == 3:
        a1, a2 = a[:, 0], a[:, 1]
        n = torch.linalg.cross(a1, a2)
        c = (beta[:, :1] * torch.linalg.cross(a2, n) + beta[:, 1:] * torch.linalg.cross(n, a1))
        c = c / (2.0 * n.square().sum(-1, keepdim=True))
    else:
        a1, a2, a3 = a[:, 0], a[:, 1], a[:, 2]
        c23 = torch.linalg.cross(a2, a3)
        c = beta[:, :1] * c23 + beta[:, 1:2] * torch.linalg.cross(a3, a1) + beta[:, 2:] * torch.linalg.cross(a1, a2)
        c = c / (2.0 * (a1 * c23).sum(-1, keepdim=True))
    return c, c.square().sum(-1) - w[:, 0]


def _empty(X, W, S, c, start, count, col):
    """AC2: no neighbour of the first vertex is nearer in power to the ortho-centre."""
    ok = torch.ones(len(S), dtype=torch.bool, device=X.device)
    step = 1 << 20
    for s in range(0, len(S), step):
        v = S[s:s + step, 0]
        row, at = _pairs(start[v], count[v])
        q = col[at]
        b = (X[q] - X[v[row]]).double()
        power = b.square().sum(1) - W[q].double() + W[v[row]].double() - 2.0 * (c[s:s + step][row] * b).sum(1)
        mine = (S[s:s + step][row] == q[:, None]).any(1)
        bad = row[(power < 0) & ~mine]
        ok[s + bad] = False
    return ok


def _extend(S, up_start, up_count, up, edges, n):
    """Rows (S, k): k above the last vertex of S and joined to every vertex."""
    out, step = [], 1 << 21
    for s in range(0, len(S), step):
        P = S[s:s + step]
        row, at = _pairs(up_start[P[:, -1]], up_count[P[:, -1]])
        k = up[at]
        keep = torch.ones(len(k), dtype=torch.bool, device=k.device)
        for v in range(P.shape[1] - 1):
            e = P[row, v] * n + k
            f = torch.searchsorted(edges, e).clamp(max=len(edges) - 1)
            keep &= edges[f] == e
        out.append(torch.cat([P[row[keep]], k[keep, None]], 1))
    return torch.cat(out) if out else torch.zeros(0, S.shape[1] + 1, dtype=torch.int64, device=S.device)


def _row_keys(R, base):
    """Ids of the distinct rows of `base`, looked up for the rows R (both sorted ascending inside a row)."""
    both = torch.cat([base, R])
    _, inv = torch.unique(both, dim=0, return_inverse=True)
    place = torch.empty(int(inv.max()) + 1, dtype=torch.int64, device=R.device)
    place[inv[:len(base)]] = torch.arange(len(base), device=R.device)
    return place[inv[len(base):]]


def _complexes(x, r, alphas):
    """[simplices, sizes] per dimension of K_alpha for every alpha."""
    n = len(r)
    X = torch.round(x * 1000.0).long()
    W = torch.round(r * 1000.0).long().square()
    aqs = [int(round(a * 1e6)) for a in alphas]
    top = max(aqs)
    i, j = _neighbours(X, W, top)
    count = torch.bincount(i, minlength=n)
    start = torch.cumsum(count, 0) - count
    S = [torch.arange(n, device=x.device)[:, None], torch.stack([i[i < j], j[i < j]], 1)]
    c, z = _centres(X, W, S[1])
    S[1] = S[1][z <= top]
    edges = S[1][:, 0] * n + S[1][:, 1]
    up_count = torch.bincount(S[1][:, 0], minlength=n)
    up_start = torch.cumsum(up_count, 0) - up_count
    for d in (2, 3):
        S.append(_extend(S[d - 1], up_start, up_count, S[1][:, 1], edges, n) if len(S[d - 1]) else
                 torch.zeros(0, d + 1, dtype=torch.int64, device=x.device))
        c, z = _centres(X, W, S[d])
        S[d] = S[d][z <= top]
    own, size, face = [], [], [None]
    for d in range(4):
        c, z = _centres(X, W, S[d])
        own.append(_empty(X, W, S[d], c, start, count, j) if len(S[d]) else torch.zeros(0, dtype=torch.bool, device=x.device))
        size.append(z)
        if d:
            f = [torch.cat([S[d][:, :k], S[d][:, k + 1:]], 1) for k in range(d + 1)]
            face.append([_row_keys(g, S[d - 1]) if d > 1 else g[:, 0] for g in f] if len(S[d]) else [])
    out = []
    for aq in aqs:
        kept, val = [None] * 4, [None] * 4
        least = None
        for d in (3, 2, 1, 0):
            ok = own[d] & (size[d] <= aq)
            v = torch.where(ok, size[d], math.inf)
            if least is not None:
                v = torch.where(ok, v, least)
            kept[d], val[d] = torch.isfinite(v), v
            if d:
                least = torch.full((len(S[d - 1]),), math.inf, dtype=torch.float64, device=x.device)
                for f in face[d]:
                    least = least.scatter_reduce(0, f, v, "amin")
        out.append([t for d in range(4) for t in (S[d][kept[d]].int(), val[d][kept[d]] / 1e6)])
    return out


def _unit(v):
    return v / v.norm(dim=-1, keepdim=True)


def _corner(v, p, r, ua, ub):
    n = (v - p) / r[:, None]
    ga = _unit(ua - (ua * n).sum(-1, keepdim=True) * n)
    gb = _unit(ub - (ub * n).sum(-1, keepdim=True) * n)
    return torch.atan2(torch.linalg.cross(ga, gb).norm(dim=-1), (ga * gb).sum(-1))


def _common(P, R):
    """Volume and boundary area of the common part of each row's balls (closed forms)."""
    k = R.shape[1]
    if k == 1:
        return 4.0 / 3.0 * math.pi * R[:, 0] ** 3, 4.0 * math.pi * R[:, 0] ** 2
    dot = lambda a, b: (a * b).sum(-1)  # noqa: E731
    if k > 2:
        e = P[:, 1:] - P[:, :1]
        h = 0.5 * (dot(e, e) - R[:, 1:] ** 2 + R[:, :1] ** 2)
        if k == 3:
            n = torch.linalg.cross(e[:, 0], e[:, 1])
            z = h[:, :1] * torch.linalg.cross(e[:, 1], n) + h[:, 1:] * torch.linalg.cross(n, e[:, 0])
            z = z / dot(n, n)[:, None]
        else:
            c23 = torch.linalg.cross(e[:, 1], e[:, 2])
            z = h[:, :1] * c23 + h[:, 1:2] * torch.linalg.cross(e[:, 2], e[:, 0]) + h[:, 2:] * torch.linalg.cross(e[:, 0], e[:, 1])
            z = z / dot(e[:, 0], c23)[:, None]
        c = P[:, 0] + z
        rho2 = R[:, 0] ** 2 - dot(z, z)
    if k == 4:
        tv = []
        for f in range(4):
            t = [v for v in range(4) if v != f]
            nt = _unit(torch.linalg.cross(P[:, t[1]] - P[:, t[0]], P[:, t[2]] - P[:, t[0]]))
            nt = torch.where((dot(nt, P[:, f] - P[:, t[0]]) < 0)[:, None], -nt, nt)
            b = dot(nt, c - P[:, t[0]])
            tv.append(c + (-b + (b * b + rho2).clamp(min=0.0).sqrt())[:, None] * nt)
    vol = area = 0.0
    for i in range(k):
        turn = flat = corner = 0.0
        for b in range(k):
            if b == i:
                continue
            dv = P[:, b] - P[:, i]
            d = dv.norm(dim=-1)
            u = dv / d[:, None]
            t = (d * d + R[:, i] ** 2 - R[:, b] ** 2) / (2 * d)
            o = P[:, i] + t[:, None] * u
            a2 = R[:, i] ** 2 - t * t
            if k == 2:
                phi, face = 2 * math.pi, math.pi * a2
            elif k == 3:
                g = P[:, 3 - i - b] - P[:, i]
                w = _unit(g - dot(g, u)[:, None] * u)
                sw = dot(c - o, w)
                cw = (a2 - sw * sw).clamp(min=1e-300).sqrt()
                half = torch.atan2(cw, sw)
                phi, face = 2 * half, a2 * half - sw * cw
            else:
                e1, f1 = [v for v in range(4) if v not in (i, b)]
                q1, q2 = tv[f1], tv[e1]
                axis = torch.where((dot(torch.linalg.cross(q1 - c, q2 - c), u) < 0)[:, None], -u, u)
                ang = torch.atan2(dot(torch.linalg.cross(q1 - o, q2 - o), axis), dot(q1 - o, q2 - o))
                phi = torch.where(ang < 0, ang + 2 * math.pi, ang)
                face = 0.5 * (a2 * phi + dot(torch.linalg.cross(o - c, q2 - q1), axis))
            flat = flat + d * face
            turn = turn + t * phi
        if k == 3:
            j, l = [v for v in range(3) if v != i]
            nrm = _unit(torch.linalg.cross(P[:, 1] - P[:, 0], P[:, 2] - P[:, 0]))
            rho = rho2.clamp(min=1e-300).sqrt()[:, None]
            uj, ul = _unit(P[:, j] - P[:, i]), _unit(P[:, l] - P[:, i])
            corner = _corner(c + rho * nrm, P[:, i], R[:, i], uj, ul) + _corner(c - rho * nrm, P[:, i], R[:, i], uj, ul)
        if k == 4:
            for f in range(4):
                if f != i:
                    j, l = [v for v in range(4) if v not in (i, f)]
                    corner = corner + _corner(tv[f], P[:, i], R[:, i], _unit(P[:, j] - P[:, i]), _unit(P[:, l] - P[:, i]))
        ai = R[:, i] ** 2 * (2 * math.pi - corner) - R[:, i] * turn
        area = area + ai
        vol = vol + (R[:, i] * ai - 0.5 * flat) / 3.0
    return vol, area


def _measure(x, r, grad):
    """Volume and area over the dual complex, and the gradient of grad . (V, A)."""
    K = _complexes(x, r, [0.0])[0]
    x, r = x.detach().clone().requires_grad_(True), r.detach().clone().requires_grad_(True)
    V = A = 0.0
    for d in range(4):
        S = K[2 * d].long()
        if len(S):
            v, a = _common(x[S], r[S])
            V, A = V + (-1.0) ** d * v.sum(), A + (-1.0) ** d * a.sum()
    (grad[0] * V + grad[1] * A).backward()
    return [torch.stack([V, A]).detach(), x.grad, r.grad]


def exact(case, seed):
    call = case["call"]
    if call == "batch" or case["n"] > 100000:
        return None
    x, r, _ = _inputs(case, seed)
    if call in ("measure", "step"):
        return _measure(x, r, torch.tensor([1.0, 0.5], dtype=torch.float64, device=x.device))
    K = _complexes(x, r, _alphas(case) if call == "sweep" else [case["alpha"]])
    K = [[t if t.is_floating_point() else None for t in k] for k in K]
    return K if call == "sweep" else K[0]
