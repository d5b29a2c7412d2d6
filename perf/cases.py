"""Workloads of the far-zone product, from the smallest call to the largest.

Each case is one call of a user's program on a plan it already holds: the
product y = T G S x of one scatterer or of a batch, in the forms the library
offers (FP32, split and single 16-bit stage 2, operators from a table or
evaluated in the kernel, trained networks in place of the operators), and
the GMRES solve that runs the product at every step. ``listed()`` names the
sizes of this repository's own workloads; ``draw(rng)`` picks another case
of the same ranges.

``exact(case, seed)`` evaluates the same product in 64 bits with plain
torch, from the definitions (free-space dyadic Green's function between the
cell-centred sites of two boxes).
"""
import math

import numpy as np
import torch

import paper_2501_04684_amd as U

TWO_PI = 2.0 * math.pi
ETA = 376.730313668


# ------------------------------------------------------------------ geometry

def _grid(nx, ny, nz):
    g = np.stack(np.meshgrid(np.arange(nx), np.arange(ny), np.arange(nz), indexing="ij"), axis=-1)
    return g.reshape(-1, 3).astype(np.int32)


def _shell(radius, thickness):
    """Boxes whose centre lies within half the thickness of the sphere of
    the given radius (both in box sides), centred on the middle box."""
    half = int(math.ceil(radius + thickness / 2))
    n = 2 * half + 1
    c = _grid(n, n, n)
    d2 = ((c - half).astype(np.float64) ** 2).sum(axis=1)
    return c[(d2 >= (radius - thickness / 2) ** 2) & (d2 < (radius + thickness / 2) ** 2)]


def _hollow(n):
    """The surface of an n x n x n cube of boxes."""
    c = _grid(n, n, n)
    return c[((c == 0) | (c == n - 1)).any(axis=1)]


def _mask(n, rho, seed):
    """About n boxes of a cube, each occupied with probability rho."""
    side = max(1, int(math.ceil((n / rho) ** (1.0 / 3.0))))
    c = _grid(side, side, side)
    keep = np.random.default_rng(seed).random(len(c)) < rho
    keep[0] = True
    return c[keep]


def _set(count, lo, hi, seed):
    """Scatterers of uneven size: shells, hollow cubes, plates, masks."""
    rng = np.random.default_rng(seed)
    out = []
    for s in range(count):
        n = float(np.exp(rng.uniform(np.log(lo), np.log(hi))))
        if s % 4 == 0:
            out.append(_shell(math.sqrt(n / (4.0 * math.pi)), 1.0))
        elif s % 4 == 1:
            out.append(_hollow(max(2, int(round(math.sqrt(n / 6.0))) + 1)))
        elif s % 4 == 2:
            thick = int(rng.integers(1, 3))
            nx = max(1, int(round(math.sqrt(n / thick * rng.uniform(1.0, 4.0)))))
            out.append(_grid(nx, max(1, int(round(n / thick / nx))), thick))
        else:
            out.append(_mask(n, rng.uniform(0.1, 1.0), int(rng.integers(1 << 31))))
    return out


def _scatterers(case):
    g = case["geometry"]
    if g == "grid":
        return [_grid(case["nx"], case["ny"], case["nz"])]
    if g == "shell":
        return [_shell(case["radius"], case["thickness"])]
    if g == "hollow":
        return [_hollow(case["side"])]
    if g == "mask":
        return [_mask(case["boxes"], case["rho"], case["place"])]
    return _set(case["count"], case["lo"], case["hi"], case["place"])


# --------------------------------------------------------------------- cases

def _case(name, geometry, **over):
    c = {"name": name, "what": "product", "geometry": geometry, "side_wl": 0.25, "n_d": 3,
         "far": "ilist", "precision": "split-fp16", "operators": "table", "basis": "identity",
         "nrhs": 1, "tuned": False}
    c.update(over)
    return c


def listed():
    return [
        # a small scatterer in the default form, one product after another:
        # the cost of a call
        _case("grid216_fp32", "grid", nx=6, ny=6, nz=6, precision="fp32"),
        # the headline product: a 4-wavelength shell with 81 basis functions
        # per box, the plan tuned once
        _case("shell3338", "shell", radius=16.0, thickness=1.0, basis="uniform", tuned=True),
        # the same in plain FP32
        _case("shell3338_fp32", "shell", radius=16.0, thickness=1.0, basis="uniform",
              precision="fp32", tuned=True),
        # several excitations of one scatterer per call
        _case("shell3338_rhs4", "shell", radius=16.0, thickness=1.0, basis="uniform", nrhs=4,
              tuned=True),
        # the shell on boxes of half the side: the basis is larger than the caches
        _case("shell25876", "shell", radius=32.0, thickness=2.0, side_wl=0.125, basis="uniform",
              tuned=True),
        # uneven boxes with testing functions of their own (not Galerkin)
        _case("hollow20_ragged_t", "hollow", side=20, basis="explicit", precision="split-bf16",
              nrhs=2),
        # a batch of scatterers with four right-hand sides, one graph per product
        _case("batch16_rhs4", "set", what="graph", count=16, lo=200, hi=20000, place=4, nrhs=4,
              tuned=True),
        # the paper's box: 4 x 4 x 4 dipoles, 192 coefficients, exact operators
        _case("sphere762_nd4", "shell", radius=8.0, thickness=1.0, side_wl=0.125, n_d=4),
        # the same with networks of 50 hidden units in place of the operators
        _case("sphere762_networks", "shell", what="networks", radius=8.0, thickness=1.0,
              side_wl=0.125, n_d=4, precision="fp32", hidden=50),
        # every pair of boxes two or more apart, without an operator table
        _case("shell3338_full", "shell", radius=16.0, thickness=1.0, far="full",
              operators="generated", basis="uniform", tuned=True),
        # one solve of a small scatterer: launches and latency
        _case("solve762", "shell", what="solve", radius=8.0, thickness=1.0, side_wl=0.25,
              precision="fp32", restart=30, tol=1e-4),
        # a solve as the serving loop runs it: random occupancy, four right-hand sides
        _case("solve5000_rhs4", "mask", what="solve", boxes=5000, rho=0.5, place=7, nrhs=4,
              precision="split-bf16", restart=30, tol=1e-4),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """Another case: any of the uses above at another size and shape."""
    what = rng.choice(["product", "product", "product", "product", "full", "graph", "networks",
                       "solve", "solve"])
    place = rng.randrange(1 << 30)
    if what == "graph":
        count = rng.randint(2, 16)
        return _case("", "set", what="graph", count=count, lo=60, hi=int(40000 / count),
                     place=place, nrhs=rng.randint(1, 4), side_wl=rng.choice([0.125, 0.25]),
                     precision=rng.choice(["split-fp16", "split-bf16", "fp32", "fp16"]),
                     n_d=rng.choice([2, 3, 3]), tuned=rng.random() < 0.5)
    n_d = rng.choice([1, 2, 3, 3, 3, 3, 4])
    lo, hi = 20, 20000
    if what == "full":
        n_d = rng.choice([1, 2, 3, 3])
        generated = rng.random() < 0.5
        hi = 2000 if generated else 600
    elif what == "networks":
        n_d = rng.choice([2, 3, 4, 4])
        hi = 4000
    elif what == "solve":
        n_d = rng.choice([2, 3, 3, 3])
        lo, hi = 200, 8000
    elif n_d == 4:
        hi = 4000
    n = _log_uniform(rng, lo, hi)
    over = {"n_d": n_d, "side_wl": rng.choice([0.125, 0.25, 0.25]), "nrhs": rng.choice([1, 1, 1, 2, 3, 4, 6])}
    if n * over["nrhs"] > 20000 or what == "full":
        over["nrhs"] = 1
    over["precision"] = "fp32" if what == "networks" else \
        rng.choice(["fp32", "split-fp16", "split-fp16", "split-bf16", "fp16"])
    geometry = rng.choice(["grid", "shell", "hollow", "mask"])
    if geometry == "grid":
        thick = rng.randint(1, 4)
        nx = max(1, int(math.sqrt(n / thick * rng.uniform(1.0, 4.0))))
        over.update(nx=nx, ny=max(1, int(n / thick / nx)), nz=thick)
    elif geometry == "shell":
        over.update(radius=math.sqrt(n / (4.0 * math.pi)), thickness=1.0)
    elif geometry == "hollow":
        over.update(side=max(2, int(math.sqrt(n / 6.0)) + 1))
    else:
        over.update(boxes=int(n), rho=rng.uniform(0.3 if what == "full" else 0.1, 1.0), place=place)
    if what == "full":
        over.update(far="full")
        if generated:
            over.update(operators="generated", precision=rng.choice(["split-fp16", "split-bf16"]))
        what = "product"
    if what == "product":
        over.update(basis=rng.choice(["identity", "uniform", "uniform", "ragged", "explicit"]),
                    tuned=rng.random() < 0.5)
        if n > 4000 and over["basis"] != "identity":
            over["nrhs"] = 1
    elif what == "networks":
        over.update(hidden=rng.randint(1, 64), nrhs=min(over["nrhs"], 2))
    elif what == "solve":
        over.update(restart=rng.choice([10, 30, 100]), tol=rng.choice([1e-3, 1e-4]),
                    basis="identity")
        if over["precision"] == "fp16":
            over["precision"] = "split-fp16"
    return _case("", geometry, what=what, **over)


# -------------------------------------------------------------------- inputs

def _functions_per_box(case, n_box, n_u):
    """N_b of every box: as many functions as coefficients, or 0 to 120."""
    if case["basis"] == "uniform":
        return np.full(n_box, n_u)
    nb = np.random.default_rng(5).integers(0, 121, size=n_box)
    nb[0] = max(nb[0], 1)
    return nb


def _normal(shape, gen, dev):
    z = torch.empty(tuple(shape) + (2,), dtype=torch.float32, device=dev)
    z.normal_(generator=gen)
    return torch.view_as_complex(z)


def _inputs(case, seed, dev, n_box, n_off):
    """The arrays a program brings: coefficients, basis, network weights."""
    n_u = 3 * case["n_d"] ** 3
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    d = {"nb_ptr": None, "S": None, "T": None}
    n = n_box * n_u
    if case["basis"] != "identity":
        nb = _functions_per_box(case, n_box, n_u)
        d["nb_ptr"] = np.concatenate([[0], np.cumsum(nb)]).astype(np.int64)
        n = int(d["nb_ptr"][-1])
        d["S"] = _normal((n_u * n,), gen, dev) / math.sqrt(n_u)
        if case["basis"] == "explicit":
            d["T"] = _normal((n_u * n,), gen, dev) / math.sqrt(n_u)
    d["x"] = _normal((case["nrhs"], n), gen, dev)
    if case["what"] == "networks":
        h = case["hidden"]
        d["net"] = (_normal((n_off, h, n_u), gen, dev) / math.sqrt(n_u),
                    _normal((n_off, h), gen, dev) * 0.1,
                    _normal((n_off, n_u, h), gen, dev) / math.sqrt(h),
                    _normal((n_off, n_u), gen, dev) * 0.1)
    return d


def _shift(case, n_box):
    """The shift of the solved system: about twice the norm of the far-zone
    product, at 45 degrees, so that the residual falls by about one half per
    step. The norm grows with the coefficients per box, the far-zone
    neighbours per box and, in wavelengths, with smaller boxes (fitted to
    power iterations on masks, shells, plates and cubes)."""
    per_box = max(1.0, _count_pairs(case) / n_box)
    size = 18000.0 * (case["n_d"] ** 3 / 27.0) * (0.25 / case["side_wl"]) ** 1.8 * per_box ** 0.7
    return complex(size * np.exp(0.25j * np.pi))


def prepare(case, seed):
    parts = _scatterers(case)
    n_box = sum(len(p) for p in parts)
    a, many = case["side_wl"], len(parts) > 1
    ff = U.FarField(None if many else parts[0], a, TWO_PI, case["n_d"], case["far"],
                    max_nrhs=case["nrhs"], precision=case["precision"],
                    scatterers=parts if many else None, operators=case["operators"])
    d = _inputs(case, seed, "cuda", n_box, ff.info["n_offsets"])
    if d["S"] is not None:
        ff.set_basis(d["nb_ptr"], d["S"], d["T"])
    state = {"what": case["what"], "ff": ff, "x": d["x"], "keep": d}
    if case["what"] == "networks":
        ff.set_networks(*d["net"])
    if case["tuned"]:
        ff.tune(case["nrhs"])
    if case["what"] == "graph":
        state["y"] = torch.empty_like(d["x"])
        ff.capture(d["x"], state["y"])
    if case["what"] == "solve":
        state["solver"] = U.Solver(ff, _shift(case, n_box), nrhs=case["nrhs"],
                                   restart=case["restart"], tol=case["tol"])
    return state


def run(state):
    if state["what"] == "graph":
        state["ff"].replay()
        return state["y"]
    if state["what"] == "solve":
        return state["solver"].solve(state["x"])[0]
    return state["ff"](state["x"])


# ---------------------------------------------------------------------- work

def _lookup(boxes):
    """Dense index of the boxes with a border of three, -1 where empty."""
    dims = boxes.max(axis=0) + 7
    at = np.full(dims, -1, dtype=np.int64)
    at[tuple((boxes + 3).T)] = np.arange(len(boxes))
    return at


def _offsets():
    w = _grid(7, 7, 7) - 3
    return w[np.abs(w).max(axis=1) >= 2]


def _pairs_of(boxes, at, w, parents=True):
    """(test, source) of every pair of boxes with offset w = c_t - c_s; with
    ``parents`` only those whose parents floor(c/2) are neighbours."""
    s = at[tuple((boxes - w + 3).T)]
    keep = s >= 0
    if parents:
        keep &= (np.abs(boxes // 2 - (boxes - w) // 2).max(axis=1) <= 1)
    t = np.nonzero(keep)[0]
    return t, s[t]


def _count_pairs(case):
    total = 0
    for boxes in _scatterers(case):
        at = _lookup(boxes)
        if case["far"] == "full":
            near = _grid(3, 3, 3) - 1
            total += len(boxes) ** 2 - sum(len(_pairs_of(boxes, at, w, False)[0]) for w in near)
        else:
            total += sum(len(_pairs_of(boxes, at, w)[0]) for w in _offsets())
    return total


def work(case):
    """One pass: the caller's arrays once each way, the multiply-adds of the
    operators (for every pair of a FULL far set at most those of a discrete
    convolution on the lattice of the sites) and of the basis."""
    parts = _scatterers(case)
    n_box = sum(len(p) for p in parts)
    n_u, nrhs = 3 * case["n_d"] ** 3, case["nrhs"]
    pairs = _count_pairs(case)
    if case["basis"] == "identity":
        n, basis = n_box * n_u, 0
    else:
        n = int(_functions_per_box(case, n_box, n_u).sum())
        basis = n * n_u
    per_pair = 16.0 * case["hidden"] * n_u if case["what"] == "networks" else 8.0 * n_u * n_u
    flops = per_pair * pairs * nrhs
    if case["far"] == "full":
        cells = float(np.prod([2.0 * case["n_d"] * s for s in parts[0].max(axis=0) + 1]))
        flops = min(flops, nrhs * cells * (6 * 5 * math.log2(cells) + 72))
    flops += 16.0 * basis * nrhs
    nbytes = 16.0 * n * nrhs + 8.0 * basis * (2 if case["basis"] == "explicit" else 1)
    if case["what"] == "networks":
        n_off = sum(1 for w in _offsets() if len(_pairs_of(parts[0], _lookup(parts[0]), w)[0]))
        nbytes += 8.0 * n_off * (2 * n_u * case["hidden"] + n_u + case["hidden"])
    if case["what"] == "solve":
        # the residual halves per step: log2(1 / tol) products and as many
        # orthogonalisations (two passes over j vectors at step j)
        steps = math.ceil(math.log2(1.0 / case["tol"]))
        flops = flops * steps + 32.0 * n * nrhs * steps * (steps + 1) / 2
    return {"bytes": nbytes, "flops": flops}


# --------------------------------------------------------------------- exact

def _green(R, k):
    """Dyadic free-space Green's function at the vectors R (..., 3): (..., 3,
    3) complex128, time convention exp(+j omega t); zero at R = 0."""
    r = R.norm(dim=-1)
    zero = r == 0
    r = torch.where(zero, torch.ones_like(r), r)
    rh = R / r[..., None]
    kr = k * r
    psi = -1j * k * ETA * torch.exp(-1j * kr) / (4.0 * math.pi * r)
    iso = psi * (1.0 - 1j / kr - 1.0 / kr ** 2)
    rr = psi * (1.0 - 3j / kr - 3.0 / kr ** 2)
    eye = torch.eye(3, dtype=R.dtype, device=R.device)
    D = eye * iso[..., None, None] - rh[..., :, None] * rh[..., None, :] * rr[..., None, None]
    return torch.where(zero[..., None, None], torch.zeros_like(D), D)


def _sites(n_d, a, dev):
    m = torch.from_numpy(_grid(n_d, n_d, n_d).astype(np.float64)).to(dev)
    return a * ((m + 0.5) / n_d - 0.5)


def _operator(w, case, dev):
    """G_w, (n_u, n_u): row (site of the test box, component)."""
    s = _sites(case["n_d"], case["side_wl"], dev)
    shift = case["side_wl"] * torch.tensor([float(v) for v in w], dtype=torch.float64, device=dev)
    D = _green(shift + s[:, None, :] - s[None, :, :], TWO_PI)
    n_u = 3 * len(s)
    return D.permute(0, 2, 1, 3).reshape(n_u, n_u)


def _far(case, dev):
    """The translation P -> E, (nrhs, boxes, n_u) complex128 both."""
    parts = _scatterers(case)
    n_box = sum(len(p) for p in parts)
    n_u = 3 * case["n_d"] ** 3

    def grouped(offsets, parents):
        starts = np.concatenate([[0], np.cumsum([len(p) for p in parts])])
        ats = [_lookup(p) for p in parts]
        out = []
        for w in offsets:
            got = [_pairs_of(p, at, w, parents) for p, at in zip(parts, ats)]
            t = np.concatenate([g[0] + s for g, s in zip(got, starts)])
            s_ = np.concatenate([g[1] + s for g, s in zip(got, starts)])
            if len(t):
                out.append((w, torch.from_numpy(t).to(dev), torch.from_numpy(s_).to(dev)))
        return out

    def products(groups, P, apply):
        E = torch.zeros_like(P)
        for i, (w, t, s) in enumerate(groups):
            for r in range(P.shape[0]):
                E[r].index_add_(0, t, apply(i, P[r].index_select(0, s)))
        return E

    if case["far"] == "full":
        # every pair of sites but those of one box or of neighbouring boxes:
        # the convolution over the common lattice of the sites, less the
        # products of the 27 near offsets
        boxes, n_d = parts[0], case["n_d"]
        near = grouped(_grid(3, 3, 3) - 1, False)
        ops = [_operator(w, case, dev) for w, _, _ in near]
        dims = [int(v) * n_d for v in boxes.max(axis=0) + 1]
        size = [2 * v for v in dims]
        axes = [torch.tensor([i if i < s // 2 else i - s for i in range(s)], dtype=torch.float64,
                             device=dev) * (case["side_wl"] / n_d) for s in size]
        R = torch.stack(torch.meshgrid(*axes, indexing="ij"), dim=-1)
        K = _green(R, TWO_PI)
        K = torch.fft.fftn(K, dim=(0, 1, 2))
        m = torch.from_numpy(_grid(n_d, n_d, n_d).astype(np.int64))
        site = torch.from_numpy(boxes.astype(np.int64))[:, None, :] * n_d + m[None]
        ix, iy, iz = (site[..., d].reshape(-1).to(dev) for d in range(3))

        def full(P):
            E = []
            for r in range(P.shape[0]):
                f = torch.zeros(size + [3], dtype=torch.complex128, device=dev)
                f[ix, iy, iz] = P[r].reshape(-1, 3)
                f = torch.fft.fftn(f, dim=(0, 1, 2))
                f = (K * f[..., None, :]).sum(-1)
                f = torch.fft.ifftn(f, dim=(0, 1, 2))
                E.append(f[ix, iy, iz].reshape(n_box, n_u))
            return torch.stack(E) - products(near, P, lambda i, v: v @ ops[i].T)
        return full

    groups = grouped(_offsets(), True)
    if case["what"] == "networks":
        def net(P, weights):
            W1, b1, W2, b2 = (t.to(torch.complex128) for t in weights)

            def apply(i, v):
                s = v.abs().amax(dim=1, keepdim=True)
                z = torch.where(s > 0, v / torch.where(s > 0, s, torch.ones_like(s)),
                                torch.zeros_like(v)) @ W1[i].T + b1[i]
                z = torch.complex(z.real.clamp(min=0), z.imag.clamp(min=0))
                return s * (z @ W2[i].T + b2[i])
            return products(groups, P, apply)
        return net
    ops = [_operator(w, case, dev) for w, _, _ in groups]
    return lambda P: products(groups, P, lambda i, v: v @ ops[i].T)


def _gmres(A, b, tol, restart, max_steps=300):
    """Restarted GMRES of every row of b from x = 0; a row stops at the step
    at which its residual estimate reaches tol."""
    out = []
    for row in b:
        x, r, bn, steps = torch.zeros_like(row), row, row.norm(), 0
        done = bool(bn == 0)
        while not done and steps < max_steps:
            beta = r.norm()
            V, H = [r / beta], np.zeros((restart + 1, restart), dtype=np.complex128)
            for j in range(restart):
                w = A(V[j])
                for _ in range(2):
                    h = torch.stack([torch.vdot(v, w) for v in V])
                    w = w - (h[:, None] * torch.stack(V)).sum(0)
                    H[:j + 1, j] += h.cpu().numpy()
                H[j + 1, j] = float(w.norm())
                V.append(w / w.norm())
                e = np.zeros(j + 2, dtype=np.complex128)
                e[0] = float(beta)
                y = np.linalg.lstsq(H[:j + 2, :j + 1], e, rcond=None)[0]
                steps += 1
                done = np.linalg.norm(e - H[:j + 2, :j + 1] @ y) <= tol * float(bn)
                if done or steps >= max_steps:
                    break
            x = x + (torch.from_numpy(y).to(x.device)[:, None] * torch.stack(V[:len(y)])).sum(0)
            if not done:
                r = row - A(x)
                done = bool(r.norm() <= tol * bn)
        out.append(x)
    return torch.stack(out)


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    parts = _scatterers(case)
    n_box, n_u = sum(len(p) for p in parts), 3 * case["n_d"] ** 3
    n_off = 0
    if case["what"] == "networks":
        n_off = sum(1 for w in _offsets() if len(_pairs_of(parts[0], _lookup(parts[0]), w)[0]))
    d = _inputs(case, seed, dev, n_box, n_off)
    far = _far(case, dev)
    x = d["x"].to(torch.complex128)
    if case["what"] == "networks":
        return far(x.reshape(-1, n_box, n_u), d["net"]).reshape(x.shape)
    if case["what"] == "solve":
        sigma = _shift(case, n_box)

        def A(v):
            return sigma * v + far(v.reshape(1, n_box, n_u)).reshape(-1)
        return _gmres(A, x, case["tol"], case["restart"])
    if case["basis"] == "identity":
        return far(x.reshape(-1, n_box, n_u)).reshape(x.shape)
    # per box: P = S x, y = T E with T = S^T unless given; the boxes of one
    # function count are taken together
    ptr = d["nb_ptr"]
    nb = np.diff(ptr)
    P = torch.zeros((x.shape[0], n_box, n_u), dtype=torch.complex128, device=dev)
    y = torch.zeros_like(x)
    groups = []
    for v in np.unique(nb[nb > 0]):
        for b in np.array_split(np.nonzero(nb == v)[0], max(1, int((nb == v).sum()) // 4096)):
            first = torch.from_numpy(ptr[b]).to(dev)
            at = first[:, None] * n_u + torch.arange(int(v) * n_u, device=dev)
            cols = first[:, None] + torch.arange(int(v), device=dev)
            groups.append((int(v), torch.from_numpy(b).to(dev), at, cols))
    for v, b, at, cols in groups:
        S = d["S"][at].to(torch.complex128).reshape(len(b), v, n_u)  # [function][coefficient]
        for r in range(x.shape[0]):
            P[r, b] = (S * x[r][cols][..., None]).sum(1)
    E = far(P)
    for v, b, at, cols in groups:
        src = d["S"] if d["T"] is None else d["T"]
        M = src[at].to(torch.complex128)
        M = M.reshape(len(b), v, n_u) if d["T"] is None else \
            M.reshape(len(b), n_u, v).transpose(1, 2)
        for r in range(x.shape[0]):
            y[r][cols] = (M * E[r, b][:, None, :]).sum(2)
    return y
