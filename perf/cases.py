"""The workloads by which the framework's speed is judged, and their ranges.

Four kinds of work, all through the package's public entry points:

* ``product``: y = A x on a resident geometry (``Geometry.matvec``), the inner
  operation of every Krylov step and of every serving request;
* ``batch``: one product on each of several resident geometries
  (``matvec_batch``), as a service with several models in memory runs them;
* ``solve``: a budget of preconditioned GMRES steps on plane-wave excitations
  (``Geometry.gmres`` with the sparse approximate inverse);
* ``setup``: a new geometry up to its first product (octree, tables, tuning,
  near-field integrals), what every new mesh costs once.

Surfaces are closed triangle meshes at about a tenth of the wavelength
(wavelength 1, k = 2 pi, quarter-wavelength leaf boxes): geodesic spheres,
ellipsoids and rounded boxes of 1 000 to 280 000 RWG functions.
"""
import math

import numpy as np
import torch

import paper_2210_04892_amd as mf
import synth

K0 = 2.0 * math.pi
LEAF = 0.25
DTYPES = {"c64": torch.complex64, "c128": torch.complex128}


def listed():
    def case(name, **more):
        return {"name": name, **more}

    return [
        # the smallest scatterer, one vector: a Krylov step whose cost is launches and latency
        case("sphere_r0.5_c64_1", kind="product", surface="sphere", m=8, size=0.5, op="C", dtype="c64", nrhs=1),
        # a small one, Stratton-Chu pair in double precision, an odd number of vectors
        case("sphere_m6_em_c128_5", kind="product", surface="sphere", m=6, size=0.5, op="EM", dtype="c128", nrhs=5),
        # a medium scatterer inside a single-vector solver, both precisions
        case("sphere_r3_c64_1", kind="product", surface="sphere", m=36, size=3.0, op="C", dtype="c64", nrhs=1),
        case("sphere_r3_c128_1", kind="product", surface="sphere", m=36, size=3.0, op="C", dtype="c128", nrhs=1),
        # a few vectors at once (two polarisations of a few angles): too many for the one-vector kernels, too few
        # for the matrix cores; an ellipsoid, whose boxes are filled unevenly
        case("ellipsoid_em_c64_7", kind="product", surface="ellipsoid", m=40, size=3.2, op="EM", dtype="c64", nrhs=7),
        # a monostatic sweep: 64 plane waves on a box with flat sides
        case("box_c64_64", kind="product", surface="box", m=55, size=4.0, op="C", dtype="c64", nrhs=64),
        # the same body with 16 vectors in double precision
        case("box_c128_16", kind="product", surface="box", m=55, size=4.0, op="C", dtype="c128", nrhs=16),
        # the largest body (552 960 unknowns), 16 vectors, both precisions
        case("sphere_r8_c64_16", kind="product", surface="sphere", m=96, size=8.0, op="C", dtype="c64", nrhs=16),
        case("sphere_r8_c128_16", kind="product", surface="sphere", m=96, size=8.0, op="C", dtype="c128", nrhs=16),
        # eight resident models of 2 300 to 64 800 RWGs, four vectors each, one call
        case("batch_8_c64_4", kind="batch", count=8, n_min=2000, n_max=150000, mesh_seed=5, op="C", dtype="c64", nrhs=4),
        # ten steps of the preconditioned solver on one excitation
        case("solve_sphere_r3_c64", kind="solve", surface="sphere", m=36, size=3.0, op="C", dtype="c64", nrhs=1,
             steps=10, pattern=16),
        # a new mesh up to its first product
        case("setup_box_c64", kind="setup", surface="box", m=24, size=1.7, op="C", dtype="c64", nrhs=4),
    ]


def draw(rng):
    """One more case of the same ranges (rng: random.Random)."""
    def between(a, b):
        return math.exp(rng.uniform(math.log(a), math.log(b)))

    kind = rng.choices(["product", "batch", "solve", "setup"], [7, 1, 1, 1])[0]
    op, dtype = rng.choice(["C", "C", "EM"]), rng.choice(["c64", "c64", "c128"])
    if kind == "batch":
        # as in the serving workload: each model's size log-uniform
        return {"kind": kind, "count": rng.randint(2, 8), "n_min": 2000, "n_max": int(between(8000, 60000)),
                "mesh_seed": rng.randint(6, 10**6), "op": op, "dtype": dtype, "nrhs": rng.randint(1, 8)}
    surface = rng.choice(["sphere", "ellipsoid", "box"])
    # frequency of the mesh: 30 m^2 RWGs (box: 9 m^2), so that all three span the same counts; new meshes and
    # solves up to the size a pass of two seconds allows
    top = {"product": 250000, "solve": 40000, "setup": 9000}[kind]
    n = between(1100, top)
    m = max(5, round(math.sqrt(n / (9 if surface == "box" else 30))))
    size = round(m * (rng.uniform(0.055, 0.074) if surface == "box" else rng.uniform(0.064, 0.083)), 4)
    case = {"kind": kind, "surface": surface, "m": m, "size": size, "op": op, "dtype": dtype}
    if kind == "product":
        # vectors: one, a few or a block, at most the work of the largest listed case
        most = max(1, min(64, int(2.4e5 * 16 / n)))
        case["nrhs"] = min(most, rng.choice([1, 1, rng.randint(2, 15), int(between(16, 64))]))
    elif kind == "solve":
        # the second-kind operator: the Stratton-Chu pair's first-kind system is not one that ten steps solve
        case.update(op="C", nrhs=rng.randint(1, 3), steps=rng.randint(5, 12), pattern=rng.choice([8, 16]))
    else:
        case["nrhs"] = rng.randint(1, 16)
    return case


# ------------------------------------------------------------------ geometry
def _mesh(case):
    m, size = case["m"], case["size"]
    if case["surface"] == "sphere":
        return synth.icosphere(m, size)
    if case["surface"] == "ellipsoid":
        return synth.ellipsoid(m, (size, 0.75 * size, 0.5 * size))
    return synth.rounded_box((size, size, 0.25 * size), 0.05 * size, size / m)


def _meshes(case):
    if case["kind"] == "batch":
        return [(v, t) for _, v, t in synth.serving_set(case["mesh_seed"], case["count"], case["n_min"], case["n_max"])]
    return [_mesh(case)]


_resident = {}


def _geometries(case):
    """The resident geometries of a case.  A program builds a geometry once and
    multiplies many vectors with it, so the last two sets stay resident."""
    shared = ("surface", "m", "size", "count", "n_min", "n_max", "mesh_seed", "pattern")
    key = tuple(case.get(f) for f in shared) + (case["nrhs"],)
    if key not in _resident:
        while len(_resident) > 1:
            _resident.pop(next(iter(_resident)))
        made = [mf.Geometry(v, t, k=K0, leaf=LEAF, max_rhs=case["nrhs"]).precompute() for v, t in _meshes(case)]
        if case["kind"] == "solve":
            made[0].sai_build(case["op"], case["pattern"])
        _resident[key] = made
    return _resident[key]


def _coefficients(n2, nrhs, dtype, seed):
    """Vectors as a Krylov iteration meets them: real and imaginary parts
    N(0, 1), one contiguous row per vector."""
    gen = torch.Generator("cuda").manual_seed(seed)
    x = torch.randn(nrhs, n2, 2, dtype=torch.float64, device="cuda", generator=gen)
    return torch.view_as_complex(x).to(dtype).t()


def prepare(case, seed):
    dtype, nrhs = DTYPES[case["dtype"]], case["nrhs"]
    if case["kind"] == "setup":
        # a new body: the case's surface, a little larger or smaller
        v, t = _mesh(case)
        v = v * (1 - 0.02 * np.random.default_rng(seed).random())
        return {"case": case, "verts": v, "tris": t, "x": _coefficients(len(t) * 3, nrhs, dtype, seed)}
    made = _geometries(case)
    state = {"case": case, "geometries": made}
    if case["kind"] == "solve":
        khat, pol = synth.plane_waves(nrhs, seed)
        state["b"] = made[0].plane_wave_rhs(khat, pol, dtype=dtype)
    else:
        state["x"] = [_coefficients(2 * g.n_rwg, nrhs, dtype, seed + 1000003 * i) for i, g in enumerate(made)]
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "setup":
        g = mf.Geometry(state["verts"], state["tris"], k=K0, leaf=LEAF, max_rhs=case["nrhs"]).precompute()
        return g.matvec(state["x"], op=case["op"])
    made = state["geometries"]
    if case["kind"] == "product":
        return made[0].matvec(state["x"][0], op=case["op"])
    if case["kind"] == "batch":
        return mf.matvec_batch([(g, x, case["op"]) for g, x in zip(made, state["x"])])
    # a fixed budget of steps (the tolerance is out of reach)
    x, _, _ = made[0].gmres(state["b"], op=case["op"], max_iters=case["steps"], tol=1e-12, precond="sai")
    return x


# ---------------------------------------------------------------------- work
def _rwg(tris):
    """(edges (N, 2) in RWG order, RWG of the edge opposite each corner (nt, 3),
    sign of its function on the triangle)."""
    a, b = tris[:, [1, 2, 0]], tris[:, [2, 0, 1]]
    pairs = np.stack([np.minimum(a, b), np.maximum(a, b)], -1).reshape(-1, 2).astype(np.int64)
    ids, back = np.unique(pairs[:, 0] * (int(tris.max()) + 1) + pairs[:, 1], return_inverse=True)
    edges = np.stack([ids // (int(tris.max()) + 1), ids % (int(tris.max()) + 1)], -1)
    return edges, back.reshape(-1, 3), np.where(a < b, 1.0, -1.0)


def _adjacent(boxes, values):
    """Sum over pairs of adjacent (or equal) boxes of values[i] values[j]."""
    key = {tuple(b): i for i, b in enumerate(boxes.tolist())}
    total = 0
    for dx in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dz in (-1, 0, 1):
                for (x, y, z), i in key.items():
                    j = key.get((x + dx, y + dy, z + dz))
                    if j is not None:
                        total += int(values[i]) * int(values[j])
    return total


def _counts(verts, tris):
    """Sizes that fix the work of one product: RWGs, near-field entries, and
    per octree level from 2 on (boxes, samples, translations)."""
    edges, _, _ = _rwg(tris)
    mid = 0.5 * (verts[edges[:, 0]] + verts[edges[:, 1]])
    lo, hi = verts.min(0), verts.max(0)
    extent = float((hi - lo).max())
    levels = max(1, int(math.ceil(math.log2(extent / LEAF) - 1e-12)) + 1)
    root = LEAF * 2 ** (levels - 1)
    at = np.clip(np.floor((mid - (0.5 * (lo + hi) - 0.5 * root)) / LEAF).astype(np.int64), 0, 2 ** (levels - 1) - 1)
    boxes, filled = np.unique(at, axis=0, return_counts=True)
    near, per_level = _adjacent(boxes, filled), []
    for level in range(levels - 1, 1, -1):
        a = LEAF * 2 ** (levels - 1 - level)
        kd = K0 * a * math.sqrt(3)
        L = math.ceil(kd + 1.8 * 3 ** (2 / 3) * kd ** (1 / 3)) + (2 if level == levels - 1 else 0)
        parents, children = np.unique(boxes // 2, axis=0, return_counts=True)
        moved = _adjacent(parents, children) - _adjacent(boxes, np.ones(len(boxes), int))
        per_level.append((len(boxes), L, 2 * (L + 1) ** 2, moved))
        boxes = parents
    return len(edges), near, per_level


def _product_work(verts, tris, nrhs, size):
    """Bytes: the vectors, the near-field entries (two per pair), both leaf
    patterns and the translation operators once each.  Operations: the
    contractions of every stage, stencils of 8 points per angle."""
    n, near, lv = _counts(verts, tris)
    total, flops = 4.0 * n * nrhs * size + 2.0 * near * size, 32.0 * near * nrhs
    for i, (count, L, samples, moved) in enumerate(lv):
        total += 316.0 * samples * size
        flops += 16.0 * moved * samples * nrhs
        if i == 0:
            total += 4.0 * n * samples * size
            flops += 64.0 * n * samples * nrhs
        else:
            below, Lc, _, _ = lv[i - 1]
            flops += 2 * below * nrhs * (64.0 * (L + 1) * (2 * Lc + 2) + 80.0 * samples)
    return total, flops


def work(case):
    size = 16 if case["dtype"] == "c128" else 8
    total = flops = 0.0
    for verts, tris in _meshes(case):
        b, f = _product_work(verts, tris, case["nrhs"], size)
        if case["kind"] == "solve":
            # a product per step and one at either end; the basis is read twice and written once per vector
            n2, s = 3.0 * len(tris), case["steps"]
            orth = n2 * case["nrhs"] * s * (s + 1)
            b, f = b * (s + 2) + orth * size, f * (s + 2) + 16 * orth
            b += s * n2 * 2 * case["pattern"] * size
        elif case["kind"] == "setup":
            # entries in both precisions and for both operator pairs; 49 point pairs of about 100 operations per
            # triangle pair of adjacent boxes, and 10^4 per region of the touching ones (13 neighbours: 24 + 15
            # regions) that share a vertex, an edge or the whole triangle
            n, near, lv = _counts(verts, tris)
            leaf = lv[0][2] if lv else 0
            b += near * 4 * 24.0 + n * leaf * 4 * 24.0
            f += near / 2.25 * 49 * 100.0 + len(tris) * 39 * 1e4 * 150.0
        total, flops = total + b, flops + f
    return {"bytes": total, "flops": flops}


# --------------------------------------------------------------------- exact
# Radon's seven points of degree 5
_S15 = math.sqrt(15.0)
_A7, _B7 = (6 - _S15) / 21, (6 + _S15) / 21
_BARY = np.array([[1 / 3] * 3] + [[c if i != j else 1 - 2 * c for i in range(3)] for c in (_A7, _B7) for j in (2, 1, 0)])
_W7 = np.array([9 / 40] + [(155 - _S15) / 1200] * 3 + [(155 + _S15) / 1200] * 3)


def _touching_rule(shared, order):
    """Points (s1, s2), (t1, t2) of two reference triangles 0 <= s2 <= s1 <= 1
    that share `shared` corners, and weights: the regularising coordinates of
    Sauter and Schwab (Boundary Element Methods, section 5.2) with Gauss rules."""
    x, w = np.polynomial.legendre.leggauss(order)
    x, w = 0.5 * (x + 1), 0.5 * w
    xi, a, b, c = (g.ravel() for g in np.meshgrid(x, x, x, x, indexing="ij"))
    wt = np.einsum("i,j,k,l->ijkl", w, w, w, w).ravel()
    if shared == 3:
        half = [((xi, xi * (1 - a + a * b)), (xi * (1 - a * b * c), xi * (1 - a))),
                ((xi, xi * a * (1 - b + b * c)), (xi * (1 - a * b), xi * a * (1 - b))),
                ((xi * (1 - a * b * c), xi * a * (1 - b * c)), (xi, xi * a * (1 - b)))]
        parts = [(p, q, xi ** 3 * a ** 2 * b) for p, q in half] + [(q, p, xi ** 3 * a ** 2 * b) for p, q in half]
    elif shared == 2:
        j = xi ** 3 * a ** 2
        parts = [((xi, xi * a * c), (xi * (1 - a * b), xi * a * (1 - b)), j),
                 ((xi, xi * a), (xi * (1 - a * b * c), xi * a * b * (1 - c)), j * b),
                 ((xi * (1 - a * b), xi * a * (1 - b)), (xi, xi * a * b * c), j * b),
                 ((xi * (1 - a * b * c), xi * a * b * (1 - c)), (xi, xi * a), j * b),
                 ((xi * (1 - a * b * c), xi * a * (1 - b * c)), (xi, xi * a * b), j * b)]
    else:
        p, q = (xi, xi * a), (xi * b, xi * b * c)
        parts = [(p, q, xi ** 3 * b), (q, p, xi ** 3 * b)]
    s = np.concatenate([np.stack(p, -1) for p, _, _ in parts])
    t = np.concatenate([np.stack(q, -1) for _, q, _ in parts])
    return s, t, np.concatenate([wt * j for _, _, j in parts])


def _kernel(r):
    """Real and imaginary parts of G = exp(-jkR) / (4 pi R) and of g with
    grad G = g (x - y)."""
    c, s, inv = torch.cos(K0 * r), torch.sin(K0 * r), 1 / (4 * math.pi * r)
    kr, i3 = K0 * r, inv / (r * r)
    return c * inv, -s * inv, -(c + kr * s) * i3, -(kr * c - s) * i3


def _touching(verts, tris, nrm, area, dev):
    """Ordered pairs of triangles that share a corner: (test, source, entries
    (pairs, 4 operators T, K, n x L, n x K, 3 test corners, 3 source corners))."""
    of = [[] for _ in range(len(verts))]
    for i, t in enumerate(tris.tolist()):
        for a in t:
            of[a].append(i)
    groups = {1: [], 2: [], 3: []}
    for i, t in enumerate(tris.tolist()):
        for j in sorted({u for a in t for u in of[a]}):
            both = [a for a in t if a in tris[j]]
            it, ij = t, tris[j].tolist()
            p = [it.index(a) for a in both] + [n for n in range(3) if it[n] not in both]
            q = [ij.index(a) for a in both] + [n for n in range(3) if ij[n] not in both]
            groups[len(both)].append((i, j, p, q))
    out = []
    V, NR, AR = (torch.as_tensor(z, device=dev) for z in (verts, nrm, area))
    for shared, found in groups.items():
        s, t, w = (torch.as_tensor(z, device=dev) for z in _touching_rule(shared, 8))
        one = torch.ones(len(w), 1, dtype=torch.float64, device=dev)
        phi, psi = torch.cat([one, s], 1), torch.cat([one, t], 1)
        basis = (phi[:, :, None] * psi[:, None, :]).reshape(-1, 9) * w[:, None]
        step = max(1, int(2e7 // len(w)))
        for at in range(0, len(found), step):
            part = found[at:at + step]
            i, j = (torch.tensor([f[n] for f in part], device=dev) for n in (0, 1))
            pi, qi = (torch.tensor([f[n] for f in part], device=dev) for n in (2, 3))
            tt, ts = torch.as_tensor(tris, device=dev).long()[i], torch.as_tensor(tris, device=dev).long()[j]
            P, Q = V[torch.gather(tt, 1, pi)], V[torch.gather(ts, 1, qi)]
            X = torch.stack([P[:, 0], P[:, 1] - P[:, 0], P[:, 2] - P[:, 1]], 1)
            Y = torch.stack([Q[:, 0], Q[:, 1] - Q[:, 0], Q[:, 2] - Q[:, 1]], 1)
            d = torch.matmul(phi, X) - torch.matmul(psi, Y)          # (pairs, points, 3)
            gr, gi, hr, hi = _kernel(d.square().sum(-1).sqrt())
            MG = torch.complex(gr @ basis, gi @ basis).reshape(-1, 3, 3)
            Mg = torch.stack([torch.complex((hr * d[..., c]) @ basis, (hi * d[..., c]) @ basis) for c in range(3)], -1)
            Mg = Mg.reshape(-1, 3, 3, 3)                             # (pairs, a, b, component)
            corner_t, corner_s = V[tt], V[ts]
            E = torch.zeros(len(part), 4, 3, 3, dtype=torch.complex128, device=dev)
            n = NR[i]
            for a in range(3):
                U = X.clone()
                U[:, 0] -= corner_t[:, a]
                TW = torch.cross(n[:, None].expand_as(U), U, dim=-1)
                for b in range(3):
                    W = Y.clone()
                    W[:, 0] -= corner_s[:, b]
                    dots = (U[:, :, None] * W[:, None]).sum(-1)
                    twd = (TW[:, :, None] * W[:, None]).sum(-1)
                    cr = torch.cross(Mg, W[:, None].expand(-1, 3, -1, -1).to(Mg.dtype), dim=-1)
                    E[:, 0, a, b] = -1j * K0 * ((MG * dots).sum((1, 2)) - 4 / K0 ** 2 * MG[:, 0, 0])
                    E[:, 1, a, b] = (U[:, :, None] * cr).sum((1, 2, 3))
                    E[:, 2, a, b] = 1j * K0 * (MG * twd).sum((1, 2)) + 2j / K0 * (TW * Mg[:, :, 0]).sum((1, 2))
                    E[:, 3, a, b] = -(TW[:, :, None] * cr).sum((1, 2, 3))
            if shared == 3:
                E[:, 1] = 0   # flat triangle: the field of its own current is normal to it
                E[:, 3] = 0
            out.append((i, j, E * (4 * AR[i] * AR[j])[:, None, None, None]))
    return out


def _dense(verts, tris, x, op, dev):
    """A x by direct summation: seven points on each triangle of a pair without
    a common corner, the regularised rules on the others."""
    nt, nrhs = len(tris), x.shape[1]
    _, of, sign = _rwg(tris)
    P = verts[tris]
    cr = np.cross(P[:, 1] - P[:, 0], P[:, 2] - P[:, 0])
    area = 0.5 * np.linalg.norm(cr, axis=1)
    nrm = cr / (2 * area)[:, None]
    length = np.linalg.norm(P[:, [1, 2, 0]] - P[:, [2, 0, 1]], axis=-1)
    coef = torch.as_tensor(sign * length / (2 * area)[:, None], device=dev)
    of = torch.as_tensor(of, device=dev)
    n = x.shape[0] // 2
    x = torch.as_tensor(x, device=dev).to(torch.complex128)
    half = torch.stack([x[:n], x[n:]], 1)                            # (N, current, rhs)
    loc = coef[:, :, None, None] * half[of]                          # (nt, corner, current, rhs)
    pts = torch.as_tensor(np.einsum("pc,tcd->tpd", _BARY, P), device=dev)
    corners = torch.as_tensor(P, device=dev)
    arm = pts[:, :, None] - corners[:, None]                         # (nt, point, corner, 3)
    wts = torch.as_tensor(_W7, device=dev)[None] * torch.as_tensor(area, device=dev)[:, None]
    cur = torch.einsum("tpcd,tckr->tpdkr", arm.to(loc.dtype), loc)
    div = 2 * loc.sum(1)[:, None].expand(-1, 7, -1, -1)
    flat = pts.reshape(-1, 3)
    jw = (cur * wts[:, :, None, None, None]).reshape(7 * nt, 3, -1)
    dw = (div * wts[:, :, None, None]).reshape(7 * nt, 1, -1)
    yd = flat[:, :, None] * dw
    yj = torch.cross(flat[:, :, None].expand(-1, -1, jw.shape[2]).to(jw.dtype), jw, dim=1)
    forG = torch.view_as_real(torch.cat([jw, dw], 1)).reshape(7 * nt, -1)
    forg = torch.view_as_real(torch.cat([jw, yj, dw, yd], 1)).reshape(7 * nt, -1)
    near = _touching(verts, tris, nrm, area, dev)
    ti, tj = torch.cat([a for a, _, _ in near]), torch.cat([b for _, b, _ in near])
    order = torch.argsort(ti)
    ti, tj = ti[order], tj[order]
    first = torch.searchsorted(ti, torch.arange(nt + 1, device=dev))
    sq = flat.square().sum(1)
    y = torch.zeros(n, 2, nrhs, dtype=torch.complex128, device=dev)
    nr = torch.as_tensor(nrm, device=dev)
    step = max(1, int(4e7 // (49 * nt)))
    for t0 in range(0, nt, step):
        t1 = min(nt, t0 + step)
        rows = flat[7 * t0:7 * t1]
        r2 = torch.addmm(sq[None] + sq[7 * t0:7 * t1, None], rows, flat.t(), alpha=-2)
        a, b = ti[first[t0]:first[t1]] - t0, tj[first[t0]:first[t1]]
        r2.view(t1 - t0, 7, nt, 7)[a, :, b] = 1.0
        gr, gi, hr, hi = _kernel(r2.sqrt_())
        for g in (gr, gi, hr, hi):
            g.view(t1 - t0, 7, nt, 7)[a, :, b] = 0.0

        def times(re, im, m):
            u, v = ((z @ m).reshape(len(rows), -1, 2, nrhs, 2) for z in (re, im))
            return torch.complex(u[..., 0] - v[..., 1], u[..., 1] + v[..., 0])

        A, phi = times(gr, gi, forG).split([3, 1], 1)
        s, ys, q, yq = times(hr, hi, forg).split([3, 3, 1, 3], 1)
        r = rows[:, :, None, None].to(s.dtype)
        E1 = torch.cross(r.expand_as(s), s, dim=1) - ys              # sum g (x - y) x J
        E2 = r * q - yq                                              # sum g (x - y) div J
        nn = nr[t0:t1].repeat_interleave(7, 0)[:, :, None, None].to(s.dtype).expand_as(s)
        F = _combine(op, -1j * K0 * A, E1, torch.cross(1j * K0 * A + 1j / K0 * E2, nn, dim=1),
                     -torch.cross(E1, nn, dim=1))
        S = _combine(op, 1j / K0 * phi, 0 * phi, 0 * phi, 0 * phi)
        if op == "C":
            J = cur[t0:t1].reshape(-1, 3, 2, nrhs)
            twist = torch.cross(nn, J, dim=1)
            F[:, :, 0] += J[:, :, 0] + 0.5 * twist[:, :, 1]
            F[:, :, 1] += 0.5 * J[:, :, 1]
        F, S = F.reshape(-1, 7, 3, 2, nrhs), S.reshape(-1, 7, 2, nrhs)
        w = wts[t0:t1]
        val = torch.einsum("tpcd,tpdkr->tckr", (arm[t0:t1] * w[:, :, None, None]).to(F.dtype), F)
        val = val + 2 * (S * w[:, :, None, None]).sum(1)[:, None]
        y.view(n, -1).index_add_(0, of[t0:t1].reshape(-1), (val * coef[t0:t1, :, None, None]).reshape(-1, 2 * nrhs))
    for i, j, E in near:
        for at in range(0, len(i), 20000):
            p, q, e = i[at:at + 20000], j[at:at + 20000], E[at:at + 20000]
            prim = [torch.matmul(e[:, o], loc[q].reshape(-1, 3, 2 * nrhs)).reshape(-1, 3, 2, nrhs) for o in range(4)]
            val = _combine(op, *(z.transpose(1, 2).reshape(-1, 2, 3, nrhs).transpose(1, 2) for z in prim))
            y.view(n, -1).index_add_(0, of[p].reshape(-1), (val * coef[p][:, :, None, None]).reshape(-1, 2 * nrhs))
    return torch.cat([y[:, 0], y[:, 1]])


def _combine(op, T, K, Tx, Kx):
    """The operator's two rows from the primitive terms of both currents (axis 2)."""
    if op == "EM":
        return torch.stack([T[:, :, 0] - K[:, :, 1], T[:, :, 1] + K[:, :, 0]], 2)
    return torch.stack([-0.5 * (T + Kx)[:, :, 0] + 0.5 * (K - Tx)[:, :, 1],
                        -0.5 * (T + Kx)[:, :, 1] + 0.5 * (Tx - K)[:, :, 0]], 2)


def exact(case, seed):
    """The dense product in double precision, where the direct sum takes
    seconds; the solver's iterate after a few steps has no such value."""
    if case["kind"] == "solve":
        return None
    out, dtype = [], DTYPES[case["dtype"]]
    for i, (v, t) in enumerate(_meshes(case)):
        if case["kind"] == "setup":
            v = v * (1 - 0.02 * np.random.default_rng(seed).random())
        points = 49.0 * len(t) ** 2
        if points > 4e10 or points * case["nrhs"] > 1.2e12:
            out.append(None)
            continue
        x = _coefficients(3 * len(t), case["nrhs"], dtype, seed + (1000003 * i if case["kind"] == "batch" else 0))
        out.append(_dense(v, t, x.cpu().numpy(), case["op"], "cuda"))
    return out if case["kind"] == "batch" else out[0]
