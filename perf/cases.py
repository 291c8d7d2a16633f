"""Performance cases: the work that a program has this library do, through its public entry points.

Surfaces are star-shaped, molecule-like closed meshes (a geodesic sphere whose
directions are scaled by a smooth random factor) at a constant vertex density,
the charges are point charges inside; sizes run from the paper's Kirkwood
sphere (320 triangles) to several hundred thousand triangles.  The kinds:

* ``apply``    one operator product of a resident mesh on device vectors (what
               every GMRES iteration does), matrix-free or by the treecode, in
               FP64 (the library's default) or FP32, first- and second-kind
               formulations;
* ``refresh``  a resident mesh set up again (geometry, Sauter-Schwab near
               field, preconditioner, and the dense matrix when the far field
               is assembled), then one product with the fresh operator;
* ``solve``    a complete solve for one charge set on a resident mesh;
* ``multi``    several charge sets on one resident mesh;
* ``batch``    one charge set on each of several resident meshes of uneven size;
* ``charges``  what depends on the charges alone: the right-hand side and the
               reaction potential at the charges from given traces.

A result of PB_FP32 or of the mixed modes is a reduced-precision result that the
C ABI hands over in double arrays; a program that asks for those modes keeps
it in single precision, and so do these cases.  PB_FP64 results stay double.
"""
import math

import numpy as np
import torch

import paper_2108_10481_amd as pbm

EPS_IN, EPS_OUT, KAPPA = 4.0, 80.0, 0.125   # the paper's constants
FORMS = {"direct": pbm.PB_DIRECT_INT, "juffer": pbm.PB_JUFFER, "muller": pbm.PB_MULLER_INT,
         "pmchwt": pbm.PB_PMCHWT_INT}
PRECS = {"none": pbm.PB_PREC_NONE, "block": pbm.PB_BLOCK_DIAG, "mass": pbm.PB_MASS, "scaled": pbm.PB_SCALED_MASS,
         "calderon": pbm.PB_CALDERON, "calderon-fast": pbm.PB_SCALED_CALDERON_INT}
PRECISION = {"fp64": pbm.PB_FP64, "fp32": pbm.PB_FP32, "bf16": pbm.PB_MIXED_BF16, "fp16": pbm.PB_MIXED_FP16}
MODES = {"free": pbm.PB_MATRIX_FREE, "assembled": pbm.PB_ASSEMBLED, "tree": pbm.PB_TREECODE}


def _case(name, kind, freq, form="direct", precision="fp64", mode="free", prec="block", kappa=KAPPA, **more):
    c = {"kind": kind, "freq": freq, "form": form, "precision": precision, "mode": mode, "prec": prec, "kappa": kappa}
    c.update(more)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the Kirkwood-size sphere of the readme and of the smoke test, default
        # options: launches and host round trips count
        _case("solve_fp64_320", "solve", 4, charges=1),
        # the library's default precision, ordinary surfaces, both kinds
        _case("apply_fp64_direct_5780", "apply", 17),
        _case("apply_fp64_juffer_12500", "apply", 25, form="juffer"),
        # the default benchmark's products: 81920 triangles direct, and a
        # medium second-kind one
        _case("apply_fp32_direct_81920", "apply", 64, precision="fp32"),
        _case("apply_fp32_juffer_20480", "apply", 32, form="juffer", precision="fp32"),
        # small single-precision surface of the serving trace's lower end
        _case("apply_fp32_muller_1620", "apply", 9, form="muller", precision="fp32"),
        # assembled far field: reassembly and one product (the sphere workload)
        _case("refresh_fp32_assembled_juffer_10580", "refresh", 23, form="juffer", precision="fp32", mode="assembled"),
        # near field and preconditioner of a large FP32 matrix-free handle
        _case("refresh_fp32_free_direct_24500", "refresh", 35, precision="fp32", only="near"),
        # 16 charge sets on one mesh in mixed BF16 (the multi-RHS workload)
        _case("multi_bf16_juffer_20480", "multi", 32, form="juffer", precision="bf16", mode="assembled", charges=50,
              sets=16),
        # uneven requests solved together (the batch workload's sizes)
        _case("batch_fp32_12", "batch", 8, precision="fp32", charges=60, requests=12, freq_max=24),
        # treecode product at a large molecule's size
        _case("apply_fp32_tree_juffer_180500", "apply", 95, form="juffer", precision="fp32", mode="tree"),
        # right-hand side and reaction potential of 2000 charges
        _case("charges_fp64_2000_40500", "charges", 45, charges=2000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["apply64", "apply32", "apply32", "tree", "refresh", "near", "solve", "multi", "batch", "charges"])
    kappa = rng.choice([KAPPA, KAPPA, round(rng.uniform(0.02, 0.4), 4), 0.0])
    form = rng.choice(["direct", "juffer", "muller", "pmchwt"])
    if kind == "apply64":
        return _case(None, "apply", _log_int(rng, 4, 36), form=form, kappa=kappa, salt=rng.randrange(1000))
    if kind == "apply32":
        return _case(None, "apply", _log_int(rng, 5, 60), form=form, precision="fp32", kappa=kappa,
                     salt=rng.randrange(1000))
    if kind == "tree":
        return _case(None, "apply", _log_int(rng, 30, 95), form=form, precision="fp32", mode="tree", kappa=KAPPA,
                     salt=rng.randrange(1000))
    if kind == "refresh":
        return _case(None, "refresh", _log_int(rng, 6, 28), form=form, precision=rng.choice(["fp32", "fp32", "fp64"]),
                     mode="assembled", kappa=kappa, salt=rng.randrange(1000))
    if kind == "near":
        return _case(None, "refresh", _log_int(rng, 8, 50), form=form, precision="fp32", only="near",
                     kappa=kappa, salt=rng.randrange(1000))
    if kind == "solve":
        form, prec, precision, mode = rng.choice([
            ("direct", "block", "fp64", "free"), ("juffer", "scaled", "fp64", "free"), ("juffer", "block", "fp32", "free"),
            ("muller", "mass", "fp32", "assembled"), ("pmchwt", "calderon", "fp32", "assembled"),
            ("pmchwt", "calderon-fast", "fp32", "assembled")])
        return _case(None, "solve", _log_int(rng, 4, 20), form=form, precision=precision, mode=mode, prec=prec,
                     kappa=KAPPA, charges=_log_int(rng, 1, 200), salt=rng.randrange(1000))
    if kind == "multi":
        return _case(None, "multi", _log_int(rng, 8, 32), form=rng.choice(["direct", "juffer"]),
                     precision=rng.choice(["bf16", "fp16"]), mode="assembled", charges=_log_int(rng, 10, 100),
                     sets=rng.randint(2, 16), salt=rng.randrange(1000))
    if kind == "batch":
        return _case(None, "batch", rng.randint(6, 9), precision=rng.choice(["fp32", "fp32", "fp64"]),
                     charges=_log_int(rng, 10, 100), requests=rng.randint(3, 16), freq_max=rng.randint(10, 20),
                     salt=rng.randrange(1000))
    return _case(None, "charges", _log_int(rng, 8, 60), charges=_log_int(rng, 5, 2000), kappa=KAPPA,
                 salt=rng.randrange(1000))


# ------------------------------------------------------------------ inputs
_SPHERES = {}


def _sphere(freq):
    """Unit geodesic sphere: 20 freq^2 triangles, counter-clockwise from outside."""
    if freq in _SPHERES:
        return _SPHERES[freq]
    g = (1.0 + math.sqrt(5.0)) / 2.0
    base = np.array([p for a in (-1.0, 1.0) for b in (-g, g) for p in ((0, a, b), (a, b, 0), (b, 0, a))], dtype=np.float64)
    dist = np.linalg.norm(base[:, None] - base[None], axis=2)
    faces = []
    for i in range(12):
        for j in range(i + 1, 12):
            for k in range(j + 1, 12):
                if max(abs(dist[i, j] - 2), abs(dist[i, k] - 2), abs(dist[j, k] - 2)) < 1e-9:
                    n = np.cross(base[j] - base[i], base[k] - base[i])
                    faces.append((i, j, k) if n @ base[i] > 0 else (i, k, j))
    ij = np.array([(i, j) for i in range(freq + 1) for j in range(freq + 1 - i)])
    at = -np.ones((freq + 2, freq + 2), dtype=np.int64)
    at[ij[:, 0], ij[:, 1]] = np.arange(len(ij))
    up = np.array([(at[i, j], at[i + 1, j], at[i, j + 1]) for i in range(freq) for j in range(freq - i)])
    down = np.array([(at[i + 1, j], at[i + 1, j + 1], at[i, j + 1]) for i in range(freq) for j in range(freq - 1 - i)],
                    dtype=np.int64).reshape(-1, 3)
    local = np.concatenate([up, down])
    w = np.stack([freq - ij.sum(1), ij[:, 0], ij[:, 1]], axis=1) / freq
    pts = np.concatenate([w @ base[list(f)] for f in faces])
    tri = np.concatenate([local + k * len(ij) for k in range(20)])
    _, first, back = np.unique(np.round(pts, 9), axis=0, return_index=True, return_inverse=True)
    xyz = pts[first] / np.linalg.norm(pts[first], axis=1, keepdims=True)
    _SPHERES[freq] = (xyz, back.reshape(-1)[tri].astype(np.int32))
    return _SPHERES[freq]


def _radius(u, wave):
    k, phase, amp = wave
    f = (np.cos(u @ k.T + phase) * amp).sum(axis=1)
    return 1.0 + 0.45 * np.tanh(f / 3.0)


def _molecule(freq, rng, ncharge):
    """A surface of 20 freq^2 triangles at the benchmark's vertex density and charges inside it."""
    u, tri = _sphere(freq)
    size = 18.0 * math.sqrt(20.0 * freq * freq / 81920.0)
    wave = (rng.normal(0.0, 2.0, (8, 3)), rng.uniform(0.0, 2.0 * math.pi, 8), rng.normal(0.0, 0.5, 8))
    xyz = u * (size * _radius(u, wave))[:, None]
    if ncharge == 0:
        return xyz, tri, None, None
    d = rng.normal(size=(ncharge, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    r = 0.8 * size * _radius(d, wave) * rng.random(ncharge) ** (1.0 / 3.0)
    return xyz, tri, d * r[:, None], rng.uniform(-1.0, 1.0, ncharge)


def _traces(xyz, rng):
    """A vector like the ones a solve multiplies: smooth potential traces with a rough part, [dirichlet; neumann]."""
    c = 0.5 * xyz[rng.integers(0, len(xyz), 8)]
    q = rng.uniform(-1.0, 1.0, 8)
    d = xyz[:, None] - c[None]
    r = np.linalg.norm(d, axis=2)
    phi = (q / r).sum(1)
    dphi = -(q * (d * xyz[:, None]).sum(2) / (r ** 3 * np.linalg.norm(xyz, axis=1)[:, None])).sum(1)
    v = np.concatenate([phi / np.linalg.norm(phi), dphi / np.linalg.norm(dphi)])
    return v + 0.2 * rng.normal(size=v.size) / math.sqrt(v.size)


def _rng(case, seed):
    return np.random.default_rng([int(seed), int(case.get("salt", 0)), int(case["freq"])])


def _options(case, form=None, **more):
    return pbm.pb_default_options(eps_in=EPS_IN, eps_out=EPS_OUT, kappa=case["kappa"], formulation=FORMS[form or case["form"]],
                                  preconditioner=PRECS[case["prec"]], precision=PRECISION[case["precision"]],
                                  operator_mode=MODES[case["mode"]],
                                  calderon_fast=1 if case["prec"] == "calderon-fast" else 0, **more)


_STREAM = []


def _stream():
    """The program's own stream, on which it hands device vectors to the library."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    return _STREAM[0]


def _requests(case, seed):
    """The batch's requests: (frequency, formulation) by turns, uneven sizes."""
    rng = _rng(case, seed)
    lo, hi = math.log(case["freq"]), math.log(case["freq_max"])
    n = case["requests"]
    freqs = [int(round(math.exp(lo + (hi - lo) * k / max(n - 1, 1)))) for k in range(n)]
    return [(f, "juffer" if k % 2 else "direct") + _molecule(f, rng, case["charges"]) for k, f in enumerate(freqs)]


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "batch":
        st["handles"], st["sets"] = [], []
        for _, form, xyz, tri, qx, q in _requests(case, seed):
            st["handles"].append(pbm.pb_mesh_create(xyz, tri, _options(case, form, far_symmetric=1)))
            st["sets"].append((qx, q))
        return st
    rng = _rng(case, seed)
    xyz, tri, qx, q = _molecule(case["freq"], rng, 0 if kind in ("apply", "refresh") else case["charges"])
    st["h"] = pbm.pb_mesh_create(xyz, tri, _options(case))
    st["q"] = (qx, q)
    if kind in ("apply", "refresh"):
        st["x"] = torch.from_numpy(_traces(xyz, rng)).cuda()
        st["y"] = torch.zeros_like(st["x"])
        torch.cuda.synchronize()
    elif kind == "multi":
        st["sets"] = [(qx, rng.uniform(-1.0, 1.0, len(q))) for _ in range(case["sets"])]
    elif kind == "charges":
        st["traces"] = _traces(xyz, rng)
    return st


def _product(st):
    h, x, y = st["h"], st["x"], st["y"]
    flags = pbm.PB_APPLY_NEAR_ONLY if st["case"].get("only") == "near" else 0
    s = _stream()
    with torch.cuda.stream(s):
        pbm.pb_mesh_apply_device(h, x.data_ptr(), y.data_ptr(), flags, s.cuda_stream)
        # the near field is FP64 in every mode
        return y.clone() if st["case"]["precision"] == "fp64" or flags else y.to(torch.float32)


def _solution(case, rs):
    """phi, dphi, dG and iterations of results, in the precision the mode computes in."""
    real = np.float64 if case["precision"] == "fp64" else np.float32
    return {"phi": np.concatenate([r["phi"] for r in rs]).astype(real),
            "dphi": np.concatenate([r["dphi"] for r in rs]).astype(real),
            "dG": np.array([r["dG"] for r in rs], dtype=real),
            "iterations": np.array([r["iterations"] for r in rs], dtype=np.int64)}


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "apply":
        return _product(st)
    if kind == "refresh":
        pbm.pb_mesh_refresh(st["h"])
        return {"y": _product(st), "pinv": pbm.pb_mesh_preconditioner(st["h"])}
    if kind == "solve":
        return _solution(case, [pbm.pb_mesh_solve(st["h"], *st["q"])])
    if kind == "multi":
        return _solution(case, pbm.pb_solve_multi(st["h"], st["sets"]))
    if kind == "batch":
        return _solution(case, pbm.pb_solve_batch(st["handles"], st["sets"]))
    b = pbm.pb_mesh_rhs(st["h"], *st["q"])
    nv = st["h"].nv
    pot = pbm.pb_mesh_reaction_potential(st["h"], st["traces"][:nv], st["traces"][nv:], st["q"][0])
    return {"rhs": b, "potential": pot}


# ------------------------------------------------------------------- work
# formula operations (FMA = 2, exp and rsqrt 1) of a point pair serving both directions
_PAIR = {"direct": 8 + 2 + 2 + 4 * 8, "juffer": 8 + 2 + 8 + 4 * 12, "muller": 8 + 2 + 8 + 4 * 12, "pmchwt": 8 + 2 + 8 + 4 * 12}


def _near(t):
    """Sauter-Schwab point pairs (order 4) of t triangles: 1 identical, 3 edge and about 9 vertex neighbours each, times ~100."""
    return t * 256.0 * (6 + 3 * 5 + 9 * 2) * 100.0


def _product_work(t, form, mode="free"):
    v = t // 2 + 2
    near = 4 * 7 * v * 8.0 * 2.7
    if mode == "tree":
        # a target triangle's 6 points against some 35 clusters of 343 proxies and its neighbours' points
        return {"bytes": near + 400.0 * t, "flops": 6.0 * t * 20000.0 * 25.0}
    return {"bytes": near + 400.0 * t, "flops": 36.0 * t * t / 2 * _PAIR[form]}


def work(case):
    kind, form = case["kind"], case["form"]
    t = 20 * case["freq"] ** 2
    v = t // 2 + 2
    if kind == "apply":
        return _product_work(t, form, case["mode"])
    if kind == "refresh":
        w = {"bytes": t * 400.0 + v * 8 * 32.0, "flops": _near(t)}
        if case["mode"] == "assembled":
            size = 8.0 if case["precision"] == "fp64" else 4.0
            w = {"bytes": w["bytes"] + 2 * 4.0 * v * v * size, "flops": w["flops"] + 36.0 * t * t / 2 * 50}
        return w
    if kind == "charges":
        n = case["charges"]
        return {"bytes": 400.0 * t, "flops": 6.0 * t * n * (16 + 18 + 6)}
    its = 12
    if kind == "batch":
        w = {"bytes": 0.0, "flops": 0.0}
        n, lo, hi = case["requests"], math.log(case["freq"]), math.log(case["freq_max"])
        for k in range(n):
            f = int(round(math.exp(lo + (hi - lo) * k / max(n - 1, 1))))
            p = _product_work(20 * f * f, "juffer" if k % 2 else "direct")
            w = {"bytes": w["bytes"] + its * p["bytes"], "flops": w["flops"] + its * p["flops"]}
        return w
    if kind == "multi":
        # the 16-bit matrix once per inner product of all sets, the 32-bit one per refinement sweep and set
        return {"bytes": its * 4.0 * v * v * 2 + 2 * case["sets"] * 4.0 * v * v * 4, "flops": its * case["sets"] * 8.0 * v * v}
    if case["mode"] == "assembled":
        return {"bytes": its * 4.0 * v * v * 4, "flops": its * 8.0 * v * v}
    p = _product_work(t, form)
    return {"bytes": its * p["bytes"], "flops": its * p["flops"]}


# ------------------------------------------------------------------ exact
# The discrete Galerkin operator in 64 bits with torch: the 6-point degree-4
# rule on triangle pairs sharing no vertex, Sauter-Schwab quadrature (4 Gauss
# points per dimension) on the others.
_A, _B = 0.445948490915964886, 0.0915762135097707435
_WA, _WB = 0.223381589678011466, 0.109951743655321868


def _rule(dev):
    bary = torch.tensor([[1 - 2 * _A, _A, _A], [_A, 1 - 2 * _A, _A], [_A, _A, 1 - 2 * _A],
                         [1 - 2 * _B, _B, _B], [_B, 1 - 2 * _B, _B], [_B, _B, 1 - 2 * _B]], dtype=torch.float64, device=dev)
    return bary, torch.tensor([_WA] * 3 + [_WB] * 3, dtype=torch.float64, device=dev)


def _system(form):
    """Rows (Laplace, Yukawa) coefficients of the blocks [[K, V], [D or K, T or V]], and the identity's."""
    e = EPS_IN / EPS_OUT
    # each row: kind of trace equation (1: K, V; 2: D, T), factor of the interior and of the exterior equation
    rows = {"direct": ((1, 1, 0), (1, 0, 1)), "juffer": ((1, 1, 1 / e), (2, 1, e)), "muller": ((1, 1, 1), (2, 1, 1)),
            "pmchwt": ((1, -1, 1), (2, -1, 1))}[form]
    out = []
    for kind, ci, ce in rows:
        h = 0.5 * (ci + ce)
        if kind == 1:    # [M/2 + K_L, -V_L], [M/2 - K_Y, e V_Y]
            out.append((1, (ci, -ce), (-ci, ce * e), (h, 0.0)))
        else:            # [-D_L, M/2 - T_L], [D_Y / e, M/2 + T_Y]
            out.append((2, (-ci, ce / e), (-ci, ce), (0.0, h)))
    return out


class _Geo:
    def __init__(self, xyz, tri, dev):
        self.x = torch.from_numpy(np.ascontiguousarray(xyz)).to(dev)
        self.tri = torch.from_numpy(np.ascontiguousarray(tri)).to(dev).long()
        p = self.x[self.tri]
        self.P = p
        cr = torch.linalg.cross(p[:, 1] - p[:, 0], p[:, 2] - p[:, 0])
        ln = cr.norm(dim=1)
        self.area, self.n = 0.5 * ln, cr / ln[:, None]
        self.curl = torch.stack([-(p[:, (k + 2) % 3] - p[:, (k + 1) % 3]) for k in range(3)], 1) / (2 * self.area)[:, None, None]
        self.bary, self.w = _rule(dev)
        self.q = torch.einsum("pk,tkc->tpc", self.bary, p)
        nv = self.x.shape[0]
        t = self.tri.shape[0]
        # ordered triangle pairs sharing a vertex
        order = torch.argsort(self.tri.reshape(-1), stable=True)
        tid = torch.div(order, 3, rounding_mode="floor")
        deg = torch.bincount(self.tri.reshape(-1), minlength=nv)
        start = torch.cumsum(deg, 0) - deg
        wide = int(deg.max())
        fan = torch.full((nv, wide), -1, dtype=torch.long, device=dev)
        pos = torch.arange(3 * t, device=dev) - start[self.tri.reshape(-1)[order]]
        fan[self.tri.reshape(-1)[order], pos] = tid
        near = fan[self.tri].reshape(t, -1)
        a = torch.arange(t, device=dev)[:, None].expand_as(near)[near >= 0]
        key = torch.unique(a * t + near[near >= 0])
        self.pt, self.ps = torch.div(key, t, rounding_mode="floor"), key % t


def _far(g, x, form, kappa):
    t, nv = g.tri.shape[0], g.x.shape[0]
    dev = g.x.device
    rows = _system(form)
    u1 = (g.bary @ x[:nv][g.tri].unsqueeze(2)).squeeze(2)
    u2 = (g.bary @ x[nv:][g.tri].unsqueeze(2)).squeeze(2)
    wt = g.w[None] * g.area[:, None]
    b1, b2 = (wt * u1).reshape(-1), (wt * u2).reshape(-1)
    curl = (x[:nv][g.tri].unsqueeze(2) * g.curl).sum(1) * g.area[:, None]
    cw = (g.w[None, :, None] * curl[:, None, :]).reshape(-1, 3)
    Y = g.q.reshape(-1, 3)
    nY = g.n.repeat_interleave(6, 0)
    Yc = Y.T.contiguous()
    nb1 = nY * b1[:, None]
    step = max(1, int(1.2e8 / (36 * t)))
    by_t = torch.argsort(g.pt)
    ptr = torch.searchsorted(g.pt[by_t].contiguous(), torch.arange(t + 1, device=dev))
    y = torch.zeros(2, t, 3, dtype=torch.float64, device=dev)
    for t0 in range(0, t, step):
        t1 = min(t, t0 + step)
        m = t1 - t0
        X, nX = g.q[t0:t1].reshape(-1, 3), g.n[t0:t1].repeat_interleave(6, 0)
        d = [X[:, c, None] - Yc[c][None] for c in range(3)]
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        ri = r2.rsqrt()
        sel = by_t[ptr[t0]:ptr[t1]]
        ri.view(m, 6, t, 6)[g.pt[sel] - t0, :, g.ps[sel], :] = 0.0
        e = torch.exp(-kappa * r2 * ri).nan_to_num(1.0)
        r3 = ri ** 3
        fy = e * (r3 + kappa * ri * ri)
        gy = e * ri
        dns = d[0] * nY[:, 0] + d[1] * nY[:, 1] + d[2] * nY[:, 2]
        del r2
        for k, (kind, first, second, _) in enumerate(rows):
            if kind == 1:
                F = (first[0] * r3 + first[1] * fy) * dns
                G = second[0] * ri + second[1] * gy
                pot = (F @ b1 + G @ b2).view(m, 6)
                W = None
            else:
                dnt = d[0] * nX[:, 0, None] + d[1] * nX[:, 1, None] + d[2] * nX[:, 2, None]
                F = -(second[0] * r3 + second[1] * fy) * dnt
                G = first[0] * ri + first[1] * gy
                pot = (F @ b2 + first[1] * kappa * kappa * ((gy @ nb1) * nX).sum(1)).view(m, 6)
                W = ((G @ cw).view(m, 6, 3) * g.w[None, :, None]).sum(1)
                del dnt
            del F, G
            out = (pot * g.w[None]) @ g.bary
            if W is not None:
                out = out + (g.curl[t0:t1] * W[:, None, :]).sum(2)
            y[k, t0:t1] = out * (g.area[t0:t1] / (4 * math.pi))[:, None]
    res = torch.zeros(2 * nv, dtype=torch.float64, device=dev)
    for k in range(2):
        res[k * nv:(k + 1) * nv].index_add_(0, g.tri.reshape(-1), y[k].reshape(-1))
    return res


def _singular_points(shared, dev):
    """(u1, u2, v1, v2, weight) of the Sauter-Schwab rule: relative coordinates on the simplex 0 <= u2 <= u1 <= 1."""
    z, wz = np.polynomial.legendre.leggauss(4)
    z, wz = torch.tensor(0.5 * (z + 1), dtype=torch.float64, device=dev), torch.tensor(0.5 * wz, dtype=torch.float64, device=dev)
    s, a, b, c = (v.reshape(-1) for v in torch.meshgrid(z, z, z, z, indexing="ij"))
    w = torch.einsum("i,j,k,l->ijkl", wz, wz, wz, wz).reshape(-1)
    one = torch.ones_like(s)
    if shared == 3:
        jac = s ** 3 * a ** 2 * b
        reg = [(one, 1 - a + a * b, 1 - a * b * c, 1 - a), (one, a * (1 - b + b * c), 1 - a * b, a * (1 - b)),
               (1 - a * b * c, a * (1 - b * c), one, a * (1 - b))]
        reg = [r for u1, u2, v1, v2 in reg for r in ((u1, u2, v1, v2, jac), (v1, v2, u1, u2, jac))]
    elif shared == 2:
        j0 = s ** 3 * a ** 2
        reg = [(one, a * c, 1 - a * b, a * (1 - b), j0), (one, a, 1 - a * b * c, a * b * (1 - c), j0 * b),
               (1 - a * b, a * (1 - b), one, a * b * c, j0 * b), (1 - a * b * c, a * b * (1 - c), one, a, j0 * b),
               (1 - a * b * c, a * (1 - b * c), one, a * b, j0 * b)]
    else:
        jac = s ** 3 * b
        reg = [(one, a, b, b * c, jac), (b, b * c, one, a, jac)]
    return tuple(torch.cat([s * r[k] for r in reg]) for k in range(4)) + (torch.cat([w * r[4] for r in reg]),)


def _near_blocks(g, kappa):
    """Per ordered near pair the 3 x 3 blocks of V_L, K_L, V_Y, K_Y: (pairs, 4, 3, 3), local vertices in stored order."""
    dev = g.x.device
    same = (g.tri[g.pt][:, :, None] == g.tri[g.ps][:, None, :])
    count = same.flatten(1).sum(1)
    out = torch.zeros(len(g.pt), 4, 3, 3, dtype=torch.float64, device=dev)
    for shared in (1, 2, 3):
        pick = torch.nonzero(count == shared).squeeze(1)
        if not len(pick):
            continue
        u1, u2, v1, v2, w = _singular_points(shared, dev)
        lam = torch.stack([1 - u1, u1 - u2, u2], 1)
        mu = torch.stack([1 - v1, v1 - v2, v2], 1)
        for part in torch.split(pick, max(1, int(4e7 / len(w)))):
            t, s, eq = g.pt[part], g.ps[part], same[part]
            k3 = torch.arange(3, device=dev)
            if shared == 3:
                ot = os = k3.expand(len(part), 3)
            elif shared == 1:      # both rotated: the common vertex first
                kt, ks = eq.any(2).long().argmax(1), eq.any(1).long().argmax(1)
                ot, os = (kt[:, None] + k3) % 3, (ks[:, None] + k3) % 3
            else:                  # the common edge first, in the test triangle's cyclic order
                free = (~eq.any(2)).long().argmax(1)
                ot = (free[:, None] + 1 + k3) % 3
                os = torch.empty_like(ot)
                for m in (0, 1):
                    os[:, m] = eq[torch.arange(len(part), device=dev), ot[:, m]].long().argmax(1)
                os[:, 2] = 3 - os[:, 0] - os[:, 1]
            Pt = torch.gather(g.P[t], 1, ot[:, :, None].expand(-1, -1, 3))
            Ps = torch.gather(g.P[s], 1, os[:, :, None].expand(-1, -1, 3))
            d = torch.einsum("gk,nkc->ngc", lam, Pt) - torch.einsum("gk,nkc->ngc", mu, Ps)
            r2 = (d * d).sum(2)
            ri = r2.rsqrt()
            ek = torch.exp(-kappa * r2 * ri)
            dn = (d * g.n[s][:, None, :]).sum(2)
            f = dn * ri ** 3
            vals = torch.stack([ri, f, ek * ri, ek * (1 + kappa * r2 * ri) * f], 1) * w
            basis = (lam[:, :, None] * mu[:, None, :]).reshape(-1, 9)
            loc = (vals.reshape(-1, len(w)) @ basis).view(len(part), 4, 3, 3) * (g.area[t] * g.area[s] / math.pi)[:, None, None, None]
            rows = torch.zeros_like(loc)
            rows.scatter_(2, ot[:, None, :, None].expand(-1, 4, -1, 3), loc)
            back = torch.zeros_like(loc)
            back.scatter_(3, os[:, None, None, :].expand(-1, 4, 3, -1), rows)
            out[part] = back
    return out


def _near_terms(g, form, kappa):
    """Near blocks of the system: (row block, column block) -> (pairs, 3, 3), the mass terms among them."""
    blk = _near_blocks(g, kappa)
    VL, KL, VY, KY = (blk[:, k] for k in range(4))
    t = g.tri.shape[0]
    key = g.pt * t + g.ps
    rev = torch.searchsorted(key, g.ps * t + g.pt)
    TL, TY = KL[rev].transpose(1, 2), KY[rev].transpose(1, 2)
    cc = torch.einsum("nkc,nlc->nkl", g.curl[g.pt], g.curl[g.ps])
    nn = (g.n[g.pt] * g.n[g.ps]).sum(1)[:, None, None]
    DL = cc * VL.sum((1, 2))[:, None, None]
    DY = cc * VY.sum((1, 2))[:, None, None] + kappa * kappa * nn * VY
    hat = (torch.ones(3, 3, dtype=torch.float64, device=g.x.device) + torch.eye(3, dtype=torch.float64, device=g.x.device)) / 12
    M = torch.where((g.pt == g.ps)[:, None, None], hat * g.area[g.pt][:, None, None], torch.zeros_like(VL))
    out = {}
    for r, (kind, first, second, mass) in enumerate(_system(form)):
        L1, Y1, L2, Y2 = (KL, KY, VL, VY) if kind == 1 else (DL, DY, TL, TY)
        out[r, 0] = mass[0] * M + first[0] * L1 + first[1] * Y1
        out[r, 1] = mass[1] * M + second[0] * L2 + second[1] * Y2
    return out


def _near_product(g, terms, x):
    nv = g.x.shape[0]
    y = torch.zeros_like(x)
    for (r, c), B in terms.items():
        v = (B @ x[c * nv:(c + 1) * nv][g.tri[g.ps]].unsqueeze(2)).squeeze(2)
        y[r * nv:(r + 1) * nv].index_add_(0, g.tri[g.pt].reshape(-1), v.reshape(-1))
    return y


def _block_diagonal(g, terms):
    """Per vertex the inverse of the 2 x 2 matrix of the four blocks' diagonal entries."""
    nv = g.x.shape[0]
    A = torch.zeros(nv, 2, 2, dtype=torch.float64, device=g.x.device)
    eq = g.tri[g.pt][:, :, None] == g.tri[g.ps][:, None, :]
    at = g.tri[g.pt][:, :, None].expand(-1, 3, 3)[eq]
    for (r, c), B in terms.items():
        A[:, r, c].index_add_(0, at, B[eq])
    det = A[:, 0, 0] * A[:, 1, 1] - A[:, 0, 1] * A[:, 1, 0]
    return torch.stack([torch.stack([A[:, 1, 1], -A[:, 0, 1]], 1), torch.stack([-A[:, 1, 0], A[:, 0, 0]], 1)], 1) / det[:, None, None]


def exact(case, seed):
    kind = case["kind"]
    t = 20 * case["freq"] ** 2
    if kind not in ("apply", "refresh", "charges"):
        return None              # a solve stops at GMRES's tolerance: there is no exact value
    if t > 45000 and (kind == "apply" or t > 60000):
        return None              # over about 20 seconds
    rng = _rng(case, seed)
    xyz, tri, qx, q = _molecule(case["freq"], rng, case["charges"] if kind == "charges" else 0)
    g = _Geo(xyz, tri, "cuda")
    v = _traces(xyz, rng)
    if kind == "charges":
        nv = len(xyz)
        X, nX = g.q.reshape(-1, 3), g.n.repeat_interleave(6, 0)
        c, w = torch.from_numpy(qx).cuda(), torch.from_numpy(q).cuda()
        x = torch.from_numpy(v).cuda()
        fD, fN = torch.zeros(len(X), dtype=torch.float64, device="cuda"), torch.zeros(len(X), dtype=torch.float64, device="cuda")
        u1, u2 = ((g.bary @ x[k * nv:(k + 1) * nv][g.tri].unsqueeze(2)).squeeze(2) * (g.w[None] * g.area[:, None]) for k in (0, 1))
        pot = []
        for k in range(0, len(q), 64):
            d = X[:, None, :] - c[None, k:k + 64]
            ri = 1 / d.norm(dim=2)
            f = -(d * nX[:, None, :]).sum(2) * ri ** 3
            fD += (ri * w[k:k + 64]).sum(1)
            fN += (f * w[k:k + 64]).sum(1)
            pot.append((ri.T @ u2.reshape(-1) - f.T @ u1.reshape(-1)) / (4 * math.pi))
            # f = dG/dn_y of 1/|x - y| at the surface point y
        b = torch.zeros(2 * nv, dtype=torch.float64, device="cuda")
        for k, fv in enumerate((fD, fN)):
            loc = ((fv.view(-1, 6) * g.w[None]) @ g.bary) * (g.area / (4 * math.pi * EPS_IN))[:, None]
            b[k * nv:(k + 1) * nv].index_add_(0, g.tri.reshape(-1), loc.reshape(-1))
        return {"rhs": b, "potential": torch.cat(pot)}
    x = torch.from_numpy(v).cuda()
    terms = _near_terms(g, case["form"], case["kappa"])
    y = _near_product(g, terms, x)
    if case.get("only") != "near":
        y = y + _far(g, x, case["form"], case["kappa"])
    if kind == "apply":
        return y
    return {"y": y, "pinv": _block_diagonal(g, terms)}
