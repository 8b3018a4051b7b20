"""The work that users of this library have it do, as cases to be timed.

A case is a dict of plain values.  listed() gives the fixed ones, draw(rng)
more of the same kinds and ranges, prepare(case, seed) what a program holds
on the GPU before the call, run(state) one pass through the package's public
entry points, work(case) the bytes and flops that a pass cannot do without,
and exact(case, seed) what run returns, in 64 bits, from plain torch.

Every input is made here from the seed alone (no other module's arithmetic),
so that a change of the library cannot change what it is given.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2109_14814_amd as ms

TWO_PI = 2.0 * math.pi
ECC = 0.0094                    # eccentricity of the Jupiter-Europa problem
MU_PULS = 2.528e-5              # mass ratio of the pulsating-frame workloads
MU_PM = 2.527e-5                # mass ratio of the position-momentum workloads
BASE_U = (0.92, 0.0, 0.0, 0.05)     # pulsating state in the middle of the unstable patch
# The counters that the method defines (Alg. 1's cells and slots, the pair
# counts of each stage, the excluded triangles, the overflow flags).  The
# others describe the hashed tables' work and may change with the contents
# of the workspace.
STAT_NAMES = ("n_entries_all", "n_cells", "n_slots", "n_cand", "n_moller", "n_degenerate", "n_outside", "n_hits",
              "n_nonfinite", "overflow")


def listed():
    return [
        # one small pair looked at by hand: a call and its results on the
        # host, where launches and the round trip are the time
        {"name": "search_64", "kind": "pair", "na": 64, "ma": 64, "nb": 64, "mb": 64, "kappa": 2.0, "to_host": True},
        # the ordinary search: both meshes rewritten in place, then searched,
        # with no host round trip (a continuation loop's step)
        {"name": "search_512", "kind": "pair", "na": 512, "ma": 512, "nb": 512, "mb": 512, "kappa": 1.5,
         "to_host": False},
        # two patches carried by F^3 and F^-3 until they are long and thin:
        # crowded cells, millions of overlapping boxes, odd vertex counts
        {"name": "search_patches", "kind": "patches", "n_theta": 2049, "n_s": 257, "kappa": 0.5, "table_log2": 24,
         "enum_shape": 1},
        # a family of uneven mesh pairs searched together, 32..1024 x 16..128
        # quads a surface
        {"name": "family_256", "kind": "batch", "pairs": 256, "sizes_seed": 0, "kappa": 1.5, "table_log2": 26},
        # the paper's search: 14 layers, 112 half-layer pairs, pruned
        {"name": "layers_14", "kind": "layers", "n_theta_u": 1024, "n_theta_s": 2048, "m_quads": 34, "n_layers": 14,
         "kappa": 1.5},
        # the vertices of a patch carried three periods, the largest call
        {"name": "map_patch", "kind": "map", "frame": "pulsating", "n": 526593, "periods": 3, "steps": 4000},
        # points of a patch and their matrices DF over a period
        {"name": "matrix_262144", "kind": "matrix", "n": 262144, "periods": 1, "steps": 4000},
        # theta derivatives of the rows of a globalized mesh, a shift per row
        {"name": "shift_rows", "kind": "shift", "n_theta": 2048, "rows": 4096, "order": 1},
        # mesh points between the samples
        {"name": "interp_65536", "kind": "interp", "n_theta": 2048, "rows": 4096, "queries": 65536},
        # points and partials of a chart near its torus
        {"name": "chart_local", "kind": "chart", "n_theta": 2048, "order": 25, "queries": 4096, "periods": 0,
         "steps": 4000},
        # the same, carried by F^3 and DF^3: what one Newton step of the
        # chart refinement evaluates
        {"name": "chart_global", "kind": "chart", "n_theta": 2048, "order": 25, "queries": 4096, "periods": 3,
         "steps": 4000},
        # the mismatch of mesh hits and its gradient, forward and backward
        {"name": "refine_128", "kind": "refine", "hits": 128, "mode": "adjoint", "steps": 4000},
    ]


def _logi(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("pair", "pair", "patches", "batch", "layers", "map", "matrix", "shift", "interp", "chart",
                       "refine"))
    if kind == "pair":
        return {"kind": kind, "na": _logi(rng, 24, 600), "ma": _logi(rng, 24, 600), "nb": _logi(rng, 24, 600),
                "mb": _logi(rng, 24, 600), "kappa": rng.choice((1.0, 1.5, 2.0)), "to_host": rng.random() < 0.5}
    if kind == "patches":
        return {"kind": kind, "n_theta": _logi(rng, 129, 2049), "n_s": _logi(rng, 33, 257),
                "kappa": rng.choice((0.5, 0.75, 1.0)), "table_log2": 0, "enum_shape": rng.choice((0, 1))}
    if kind == "batch":
        return {"kind": kind, "pairs": _logi(rng, 5, 200), "sizes_seed": rng.randrange(1 << 20),
                "kappa": rng.choice((1.0, 1.5, 2.0)), "table_log2": 0}
    if kind == "layers":
        return {"kind": kind, "n_theta_u": _logi(rng, 100, 1024), "n_theta_s": _logi(rng, 100, 2048),
                "m_quads": rng.randint(8, 34), "n_layers": rng.randint(2, 14), "kappa": rng.choice((1.0, 1.5, 2.0))}
    if kind == "map":
        return {"kind": kind, "frame": rng.choice(("pulsating", "position-momentum")), "n": _logi(rng, 100, 500000),
                "periods": rng.choice((1, 2, 3, -1, -2, -3)), "steps": _logi(rng, 500, 4000)}
    if kind == "matrix":
        return {"kind": kind, "n": _logi(rng, 100, 250000), "periods": rng.choice((1, -1)),
                "steps": _logi(rng, 500, 4000)}
    if kind == "shift":
        return {"kind": kind, "n_theta": 1 << rng.randint(6, 11), "rows": _logi(rng, 10, 4096),
                "order": rng.choice((0, 1, 2))}
    if kind == "interp":
        return {"kind": kind, "n_theta": _logi(rng, 33, 2048), "rows": _logi(rng, 10, 4096),
                "queries": _logi(rng, 50, 65536)}
    if kind == "chart":
        return {"kind": kind, "n_theta": 1 << rng.randint(6, 11), "order": rng.randint(3, 25),
                "queries": _logi(rng, 20, 4096), "periods": rng.choice((0, 0, 1, 2, 3, -2, -3)),
                "steps": _logi(rng, 500, 4000)}
    return {"kind": kind, "hits": _logi(rng, 5, 500), "mode": rng.choice(("adjoint", "tangent")),
            "steps": _logi(rng, 500, 4000)}


# ------------------------------------------------------------------ inputs

def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64).to("cuda")


def _surface(c, th, s):
    """The torus-like surface ((1 + 0.3 s) cos th, (1 + 0.3 s) sin th,
    s cos(2 th + phi), s sin(th + psi)) with five modes of noise, at the
    columns th and rows s."""
    th, s = torch.broadcast_tensors(th[None, :], s[:, None])
    r = 1.0 + 0.3 * s
    out = torch.stack((r * torch.cos(th), r * torch.sin(th), s * torch.cos(2.0 * th + c["phi"]),
                       s * torch.sin(th + c["psi"])), dim=-1)
    for comp in range(4):
        for m in range(5):
            out[..., comp] += 0.002 * c["alpha"][comp, m] * torch.cos((m + 1) * th + c["gamma"][comp, m] * s
                                                                      + c["beta"][comp, m])
    return out.contiguous()


def _coeffs(rng):
    return {"phi": float(rng.uniform(0, TWO_PI)), "psi": float(rng.uniform(0, TWO_PI)),
            "alpha": rng.uniform(-1, 1, (4, 5)), "beta": rng.uniform(0, TWO_PI, (4, 5)),
            "gamma": rng.uniform(-math.pi, math.pi, (4, 5))}


def _torus(n, m, c):
    """(vertices, theta, s, periodic) of an n x m-quad surface."""
    theta, s = TWO_PI * np.arange(n) / n, np.arange(m + 1) / m
    return _surface(c, _dev(theta), _dev(s)), theta, s, True


def _pair_grids(case, seed):
    rng = np.random.default_rng(seed)
    a, b = _coeffs(rng), _coeffs(rng)
    return [(_torus(case["na"], case["ma"], a), _torus(case["nb"], case["mb"], b))]


def _batch_sizes(case):
    """Quads per surface, log-uniform in 32..1024 x 16..128."""
    rng = np.random.default_rng(case["sizes_seed"])
    pick = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    return [(pick(32, 1024), pick(16, 128), pick(32, 1024), pick(16, 128)) for _ in range(case["pairs"])]


def _batch_grids(case, seed):
    rng = np.random.default_rng(seed)
    a, b = _coeffs(rng), _coeffs(rng)
    out = []
    for i, (na, ma, nb, mb) in enumerate(_batch_sizes(case)):
        step = {"phi": 1e-3 * i, "psi": 1e-3 * i}
        ca, cb = ({**c, **{k: c[k] + v for k, v in step.items()}} for c in (a, b))
        out.append((_torus(na, ma, ca), _torus(nb, mb, cb)))
    return out


LAM, DOM = 1.35, 0.05           # multiplier and fundamental domain of the layered meshes


def _layer_s(first, last, m_quads):
    """s samples with the boundaries DOM LAM^n, n = first - 1 .. last, among
    them, m_quads quads a half-layer, and 4 quads between the innermost."""
    b = [DOM * LAM ** n for n in range(first - 1, last + 1)]
    pos = np.concatenate([[b[0]]] + [np.linspace(b[n - 1], b[n], m_quads + 1)[1:] for n in range(1, len(b))])
    return np.concatenate([-pos[::-1], np.linspace(-b[0], b[0], 5)[1:-1], pos])


def _layer_grids(case, seed):
    """The unstable and the stable mesh: one surface, the stable one
    displaced so that the two cross at points of every half-layer."""
    rng = np.random.default_rng(seed)
    c, shift = _coeffs(rng), float(rng.uniform(0, TWO_PI))
    out = []
    for n_theta, first in ((case["n_theta_u"], 1), (case["n_theta_s"], 0)):
        theta, s = TWO_PI * np.arange(n_theta) / n_theta, _layer_s(first, case["n_layers"], case["m_quads"])
        v = _surface(c, _dev(theta), _dev(s / np.max(np.abs(s))))
        if first == 0:
            ell = np.log(np.maximum(np.abs(s), 1e-300) / DOM) / math.log(LAM)
            v[..., 2] += 0.05 * torch.sin(2.0 * _dev(theta)[None, :] - shift)
            v[..., 3] += 0.05 * torch.cos(TWO_PI * _dev(ell)[:, None])
        out.append((v, theta, s, True))
    return out


def _dirs(rng):
    g = rng.standard_normal((2, 4))
    d1 = g[0] / np.linalg.norm(g[0])
    d2 = g[1] - (g[1] @ d1) * d1
    return d1, d2 / np.linalg.norm(d2)


def _patch(base, d1, d2, al, be):
    base, d1, d2 = (torch.as_tensor(x, dtype=torch.float64, device="cuda") for x in (base, d1, d2))
    return base + al[None, :, None] * d1 + be[:, None, None] * d2


def _field_puls(y, f, mu, e):
    x, v, p, q = y
    w = 1.0 / (1.0 + e * math.cos(f))
    d1, d2, v2 = x + mu, x - (1.0 - mu), v * v
    g1, g2 = (1.0 - mu) * (d1 * d1 + v2) ** -1.5, mu * (d2 * d2 + v2) ** -1.5
    return torch.stack((p, q, 2.0 * q + w * (x - g1 * d1 - g2 * d2), -2.0 * p + w * (v - (g1 + g2) * v)))


def _kepler(t, e):
    """Separation and rate of the true anomaly at time t (periapse at 0)."""
    E = t
    for _ in range(60):
        E -= (E - e * math.sin(E) - t) / (1.0 - e * math.cos(E))
    rho = 1.0 - e * math.cos(E)
    return rho, math.sqrt(1.0 - e * e) / (rho * rho)


def _field_pm(y, t, mu, e):
    x, v, p, q = y
    rho, n = _kepler(t, e)
    d1, d2, v2 = x + mu * rho, x - (1.0 - mu) * rho, v * v
    g1, g2 = (1.0 - mu) * (d1 * d1 + v2) ** -1.5, mu * (d2 * d2 + v2) ** -1.5
    return torch.stack((p + n * v, q - n * x, n * q - g1 * d1 - g2 * d2, -n * p - (g1 + g2) * v))


def _rk4(field, y, periods, mu, e, steps=96):
    """A plain fourth-order flow: good enough to make a mesh of, cheap."""
    h = (TWO_PI if periods > 0 else -TWO_PI) / steps
    for i in range(abs(periods) * steps):
        t = (i % steps) * h
        k1 = field(y, t, mu, e)
        k2 = field(y + (0.5 * h) * k1, t + 0.5 * h, mu, e)
        k3 = field(y + (0.5 * h) * k2, t + 0.5 * h, mu, e)
        k4 = field(y + h * k3, t + h, mu, e)
        y = y + (h / 6.0) * (k1 + 2.0 * (k2 + k3) + k4)
    return y


def _patch_grids(case, seed):
    """An unstable patch under F^3 and the stable patch centred where one of
    its points goes, under F^-3: the two meet there."""
    rng = np.random.default_rng(seed)
    (u1, u2), (s1, s2) = _dirs(rng), _dirs(rng)
    root = rng.uniform(-5e-4, 5e-4, 2)
    pt = np.asarray(BASE_U) + root[0] * u1 + root[1] * u2
    centre = _rk4(_field_puls, _dev(pt)[:, None], 6, MU_PULS, ECC)[:, 0]
    al, be = np.linspace(-1e-3, 1e-3, case["n_theta"]), np.linspace(-1e-3, 1e-3, case["n_s"])
    out = []
    for base, d1, d2, periods in ((BASE_U, u1, u2, 3), (centre, s1, s2, -3)):
        v = _patch(base, d1, d2, _dev(al), _dev(be))
        y = _rk4(_field_puls, v.reshape(-1, 4).T.contiguous(), periods, MU_PULS, ECC)
        out.append((y.T.contiguous().reshape(v.shape), al, be, False))
    return [tuple(out)]


def _to_pm(z):
    """Pulsating states at periapse in the position-momentum frame."""
    n0 = math.sqrt(1.0 - ECC * ECC) / (1.0 - ECC) ** 2
    q, v = (1.0 - ECC) * z[..., :2], (1.0 - ECC) * n0 * z[..., 2:]
    return torch.cat((q, v + n0 * torch.stack((-q[..., 1], q[..., 0]), dim=-1)), dim=-1).contiguous()


def _states(case, seed):
    """The points of a patch of 2e-3 around the unstable base, in the order
    of its grid."""
    d1, d2 = _dirs(np.random.default_rng(seed))
    n, cols = case["n"], min(2049, case["n"])
    z = _patch(BASE_U, d1, d2, torch.linspace(-1e-3, 1e-3, cols, dtype=torch.float64, device="cuda"),
               torch.linspace(-1e-3, 1e-3, -(-n // cols), dtype=torch.float64, device="cuda")).reshape(-1, 4)[:n]
    return z.contiguous() if case.get("frame") == "pulsating" else _to_pm(z)


def _rows(case, seed):
    """Closed curves: a base point and twelve decaying modes per row."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, modes = case["n_theta"], 12
    th = TWO_PI * torch.arange(n, dtype=torch.float64, device="cuda") / n
    k = torch.arange(modes, dtype=torch.float64, device="cuda")
    basis = torch.cat((torch.cos(k[:, None] * th), torch.sin(k[:, None] * th)))
    amp = (0.1 / (1.0 + k) ** 2).repeat(2)
    a = torch.randn((case["rows"], 4, 2 * modes), dtype=torch.float64, device="cuda", generator=g) * amp
    rows = (a.reshape(-1, 2 * modes) @ basis).reshape(case["rows"], 4, n).transpose(1, 2)
    rows = rows + 1e-3 * torch.randn(rows.shape, dtype=torch.float64, device="cuda", generator=g) / n
    return (rows + torch.tensor(BASE_U, dtype=torch.float64, device="cuda")).contiguous()


def _chart_inputs(case, seed):
    rng = np.random.default_rng(seed)
    n, order, nq = case["n_theta"], case["order"], case["queries"]
    th = TWO_PI * np.arange(n) / n
    coeffs = np.zeros((order + 1, n, 4))
    coeffs[0] = _to_pm(_dev(BASE_U)).cpu().numpy()
    for k in range(order + 1):
        for q in range(8):
            amp = (1e-3 if k == 0 else 1e-2 / (k + 1) ** 2) / (1 + q) ** 2
            c, s = rng.standard_normal((2, 4))
            coeffs[k] += amp * (np.cos(q * th)[:, None] * c + np.sin(q * th)[:, None] * s)
    m = case["periods"]
    omega, lam = (0.61, LAM) if m >= 0 else (0.47, 1.0 / LAM)
    s_max = 0.05 * (lam ** m if m else 1.0)
    return _dev(coeffs), _dev(rng.uniform(0, TWO_PI, nq)), _dev(rng.uniform(-s_max, s_max, nq)), omega, lam


def _refine_inputs(case, seed):
    """Hits with a stable patch each, centred where F^6 takes the planted
    point, and parameters a patch's width off the root (closer, f cancels
    and its last digits are rounding)."""
    rng = np.random.default_rng(seed)
    K = case["hits"]
    (u1, u2), (s1, s2) = _dirs(rng), _dirs(rng)
    stars = rng.uniform(-5e-4, 5e-4, (K, 2))
    pts = np.asarray(BASE_U) + stars[:, :1] * u1 + stars[:, 1:] * u2
    centre = _rk4(_field_puls, _dev(pts).T.contiguous(), 6, MU_PULS, ECC).T.cpu().numpy()
    U = np.concatenate([np.asarray(BASE_U), u1, u2])[None, :].repeat(K, 0)
    S = np.concatenate([centre, s1[None, :].repeat(K, 0), s2[None, :].repeat(K, 0)], axis=1)
    x = np.concatenate([stars, np.zeros((K, 2))], axis=1) + rng.uniform(-1e-3, 1e-3, (K, 4))
    return _dev(x), _dev(U), _dev(S)


# ------------------------------------------------------------ prepare, run

def _params(A, B, case, flags=0):
    p = ms.default_params(A, B, case["kappa"])
    p.table_log2, p.enum_shape, p.flags = case.get("table_log2", 0), case.get("enum_shape", 0), flags
    return p


HITS_CAP = {"pair": 1 << 10, "patches": 1 << 14, "batch": 1 << 16, "layers": 1 << 16}


def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "case": case}
    if kind in ("pair", "patches"):
        (a, b), = (_pair_grids if kind == "pair" else _patch_grids)(case, seed)
        A, B = ms.Mesh(*a), ms.Mesh(*b)
        s = ms.Searcher(A, B, _params(A, B, case), hits_cap=HITS_CAP[kind], cand_cap=1 << 20)
        s.run()                 # grows the buffers to what this pair needs
        s.hits.zero_()
        st.update(A=A, B=B, s=s)
    elif kind == "batch":
        pairs = [(ms.Mesh(*a), ms.Mesh(*b)) for a, b in _batch_grids(case, seed)]
        b = ms.Batch(pairs, [_params(x, y, case) for x, y in pairs], hits_cap=HITS_CAP[kind], cand_cap=1 << 22)
        b.run_checked(True)
        b.hits.zero_()
        st.update(b=b)
    elif kind == "layers":
        u, s = _layer_grids(case, seed)
        ls = ms.LayerSearch(ms.Mesh(*u), ms.Mesh(*s), DOM, LAM, DOM, 1.0 / LAM, case["n_layers"],
                            kappa=case["kappa"], hits_cap=HITS_CAP[kind])
        ls.run(True)
        ls.batch.hits.zero_()
        st.update(b=ls.batch, ls=ls)
    elif kind == "map":
        x = _states(case, seed)
        st.update(x=x, out=torch.empty_like(x))
    elif kind == "matrix":
        st.update(x=_states(case, seed))
    elif kind == "shift":
        rows = _rows(case, seed)
        rho = np.random.default_rng(seed).uniform(-math.pi, math.pi, case["rows"])
        st.update(rows=rows, rho=_dev(rho), out=torch.empty_like(rows))
    elif kind == "interp":
        rng = np.random.default_rng(seed)
        st.update(rows=_rows(case, seed),
                  at=torch.tensor(rng.integers(0, case["rows"], case["queries"]), device="cuda"),
                  theta=_dev(rng.uniform(0, TWO_PI, case["queries"])))
    elif kind == "chart":
        coeffs, theta, s, omega, lam = _chart_inputs(case, seed)
        st.update(chart=ms.FourierTaylor(coeffs), theta=theta, s=s, omega=omega, lam=lam)
    else:
        x, U, S = _refine_inputs(case, seed)
        st.update(x=x, U=U, S=S, e=torch.tensor(ECC, dtype=torch.float64, device="cuda"))
    return st


def _buffers(hits, stats):
    """A search's device buffers as its caller reads them: the records'
    triangles and pair, their values, and the counters."""
    return {"tri": hits.view(torch.int32).view(-1, 30)[:, :3], "values": hits.view(torch.float64).view(-1, 15)[:, 2:],
            "counts": stats.view(torch.int64)[1:11]}


def run(st):
    kind, case = st["kind"], st["case"]
    if kind in ("pair", "patches"):
        s = st["s"]
        if case.get("to_host"):
            s.run()
            hits, stats, _ = s.results()
            return {**_buffers(s.hits, s.stats), "found": len(hits), "counters": [stats[k] for k in STAT_NAMES]}
        st["A"].update()
        st["B"].update()
        s.run_async()
        return _buffers(s.hits, s.stats)
    if kind in ("batch", "layers"):
        b = st["b"]
        b.run(True)
        return {**_buffers(b.hits, b.stats), "offsets": b.offsets}
    if kind == "map":
        f, mu = (ms.propagate, MU_PULS) if case["frame"] == "pulsating" else (ms.pertbp_map, MU_PM)
        return f(st["x"], mu, ECC, case["steps"], case["periods"], out=st["out"])
    if kind == "matrix":
        return ms.pertbp_map_stm(st["x"], MU_PM, ECC, case["steps"], case["periods"])
    if kind == "shift":
        return ms.theta_shift(st["rows"], st["rho"], case["order"], out=st["out"])
    if kind == "interp":
        return ms.theta_interp(st["rows"], st["at"], st["theta"])
    if kind == "chart":
        if case["periods"] == 0:
            return st["chart"].partials(st["theta"], st["s"])
        return st["chart"].partials(st["theta"], st["s"], case["periods"], st["omega"], st["lam"], MU_PM, ECC,
                                    case["steps"])
    if case["mode"] == "adjoint":
        x, e = st["x"].detach().requires_grad_(True), st["e"].detach().requires_grad_(True)
        r = ms.mismatch_r(x, e, st["U"], st["S"], MU_PULS, case["steps"], 3, -3)
        r.sum().backward()
        return {"r": r.detach(), "grad": x.grad, "grad_e": e.grad}
    out = ms.refine_grad(st["x"], st["U"], st["S"], ms.MapParams(MU_PULS, ECC, case["steps"], 3),
                         ms.MapParams(MU_PULS, ECC, case["steps"], -3), ms.MS_REFINE_TANGENT)
    return {k: out[k] for k in ("f", "r", "grad", "J")}


# ------------------------------------------------------------------- work

# A step of the 11-stage method: 396 flops of stage sums and 28 (pulsating)
# or 30 (position-momentum) per stage of the field; four tangent columns add
# 75 per stage and 1584 of sums.
STEP_PULS, STEP_PM, STEP_MATRIX = 396 + 11 * 28, 396 + 11 * 30, 396 + 11 * 30 + 11 * 75 + 1584


def _vertices(case):
    kind = case["kind"]
    if kind == "pair":
        return case["na"] * (case["ma"] + 1) + case["nb"] * (case["mb"] + 1)
    if kind == "patches":
        return 2 * case["n_theta"] * case["n_s"]
    if kind == "batch":
        return sum(na * (ma + 1) + nb * (mb + 1) for na, ma, nb, mb in _batch_sizes(case))
    # every half-layer of the two meshes takes part in 4 pairs of a layer (a
    # stable one in the pairs of two layers)
    return 4 * case["n_layers"] * (case["m_quads"] + 1) * 2 * (case["n_theta_u"] + case["n_theta_s"])


def work(case):
    kind = case["kind"]
    if kind in HITS_CAP:
        # every vertex read once; a box (12 comparisons a triangle, two
        # triangles a vertex) and a cell (8 flops) of each
        n = _vertices(case)
        return {"bytes": 32.0 * n, "flops": 32.0 * n}
    if kind in ("map", "matrix"):
        steps = float(case["n"]) * abs(case["periods"]) * case["steps"]
        if kind == "matrix":
            return {"bytes": 192.0 * case["n"], "flops": steps * STEP_MATRIX}
        return {"bytes": 64.0 * case["n"], "flops": steps * (STEP_PULS if case["frame"] == "pulsating" else STEP_PM)}
    if kind == "shift":
        n, r = case["n_theta"], case["rows"]
        return {"bytes": 64.0 * n * r + 8.0 * r, "flops": r * 2.0 * (2 * 5 * n * math.log2(n) + 6 * n)}
    if kind == "interp":
        n, q = case["n_theta"], case["queries"]
        return {"bytes": 32.0 * n * min(case["rows"], q) + 48.0 * q, "flops": q * n * 12.0}
    if kind == "chart":
        n, q, p = case["n_theta"], case["queries"], case["order"] + 1
        steps = float(q) * abs(case["periods"]) * case["steps"]
        return {"bytes": 32.0 * n * p + 112.0 * q, "flops": q * n * (16.0 * p + 30.0) + steps * STEP_MATRIX}
    # both sides' trajectories forward, then backward at three times a
    # forward step (recomputed, and the transposed products); or five
    # tangent columns a hit, two and a half a side
    steps = 2.0 * case["hits"] * 3 * case["steps"]
    if case["mode"] == "adjoint":
        return {"bytes": case["hits"] * (32.0 + 192.0 + 48.0), "flops": steps * STEP_PULS * 4}
    return {"bytes": case["hits"] * (32.0 + 192.0 + 240.0), "flops": steps * (STEP_PULS + 3 * (396 + 11 * 20))}


# ------------------------------------------------------------------ exact

def _gbs(field, y, periods, mu, e, per_period=48, columns=8):
    """The flow by extrapolated midpoint steps (Gragg, Bulirsch and Stoer),
    order 16: much closer to the flow than the fixed-step method's error."""
    sign = 1.0 if periods > 0 else -1.0
    H = sign * TWO_PI / per_period
    ns = [2 * (j + 1) for j in range(columns)]
    for i in range(abs(periods) * per_period):
        t = (i % per_period) * H
        f0 = field(y, t, mu, e)
        row = []
        for j, n in enumerate(ns):
            h = H / n
            a, b = y, y + h * f0
            for k in range(1, n):
                a, b = b, a + (2.0 * h) * field(b, t + k * h, mu, e)
            new = [0.5 * (a + b + h * field(b, t + H, mu, e))]
            for k in range(1, j + 1):
                new.append(new[k - 1] + (new[k - 1] - row[k - 1]) * (1.0 / ((ns[j] / ns[j - k]) ** 2 - 1.0)))
            row = new
        y = row[-1]
    return y


TINY = 1e-30                    # imaginary step: the derivative with no difference taken


def _flow_jet(field, y, dys, periods, mu, e):
    """The flow of y (n, 4) and of its derivatives along each of dys."""
    n = y.shape[0]
    z = torch.cat([torch.complex(y, TINY * d) for d in dys])
    z = _gbs(field, z.T.contiguous(), periods, mu, e).T.reshape(len(dys), n, 4)
    return z[0].real.contiguous(), [w.imag / TINY for w in z]


def _spectra(rows):
    """(rows, n, 2): spectra of x + i y and px + i py over n, and the signed
    frequencies."""
    n = rows.shape[-2]
    z = torch.view_as_complex(rows.reshape(*rows.shape[:-1], 2, 2).contiguous())
    k = torch.arange(n, dtype=torch.float64, device="cuda")
    return torch.fft.fft(z, dim=-2) / n, torch.where(2 * k > n, k - n, k)


def _shifted(rows, rho, order):
    n = rows.shape[-2]
    z, k = _spectra(rows)
    ph = k[None, :] * rho[:, None]
    m = torch.complex(torch.cos(ph), torch.sin(ph)) * (1j * k) ** order
    if n % 2 == 0:
        h = n / 2
        m[:, n // 2] = (torch.cos(h * rho), -h * torch.sin(h * rho), -h * h * torch.cos(h * rho))[order] + 0j
    return torch.view_as_real(torch.fft.ifft(z * m[..., None] * n, dim=-2)).reshape(rows.shape)


def _modes(theta, n, k):
    """e^{i k theta} per query, the cosine mode at n / 2."""
    ph = theta[:, None] * k
    m = torch.complex(torch.cos(ph), torch.sin(ph))
    if n % 2 == 0:
        m[:, n // 2] = torch.cos(theta * (n / 2)) + 0j
    return m


def _interpolated(rows, at, theta):
    n = rows.shape[1]
    z, k = _spectra(rows)
    out = []
    for q in range(0, len(theta), 2048):
        m = _modes(theta[q:q + 2048], n, k)
        out.append(torch.view_as_real((z[at[q:q + 2048]] * m[..., None]).sum(1)).reshape(-1, 4))
    return torch.cat(out)


def _chart_local(coeffs, theta, s):
    n, order = coeffs.shape[1], coeffs.shape[0] - 1
    z, k = _spectra(coeffs)
    m = _modes(theta, n, k)
    ik = 1j * k
    if n % 2 == 0:
        ik[n // 2] = 0          # the derivative is taken at the samples, where this mode has none
    flat = z.permute(1, 0, 2).reshape(n, -1)
    val, der = ((w @ flat).reshape(len(theta), order + 1, 2) for w in (m, m * ik))
    p = torch.arange(order + 1, dtype=torch.float64, device="cuda")
    pw = s[:, None] ** p
    dpw = p * s[:, None] ** torch.clamp(p - 1, min=0)
    real = lambda a, w: torch.view_as_real((a * w[..., None]).sum(1)).reshape(-1, 4)  # noqa: E731
    return real(val, pw), real(der, pw), real(val, dpw)


def _exact_chart(case, seed):
    coeffs, theta, s, omega, lam = _chart_inputs(case, seed)
    m = case["periods"]
    if m == 0:
        return _chart_local(coeffs, theta, s)
    sc = lam ** -m
    w, dth, ds = _chart_local(coeffs, theta - m * omega, sc * s)
    w, (dth, ds) = _flow_jet(_field_pm, w, [dth, sc * ds], m, MU_PM, ECC)
    return w, dth, ds


def _exact_refine(case, seed):
    x, U, S = _refine_inputs(case, seed)
    K = x.shape[0]
    ends, ders = [], []
    for side, (P, m) in enumerate(((U, 3), (S, -3))):
        b, d1, d2 = P[:, :4], P[:, 4:8], P[:, 8:]
        y = b + x[:, 2 * side, None] * d1 + x[:, 2 * side + 1, None] * d2
        z = torch.cat([torch.complex(y, TINY * d) for d in (d1, d2, torch.zeros_like(y))])
        e = torch.full((3 * K,), ECC, dtype=torch.complex128, device="cuda")
        e[2 * K:] += 1j * TINY
        z = _gbs(_field_puls, z.T.contiguous(), m, MU_PULS, e).T.reshape(3, K, 4)
        ends.append(z[0].real)
        ders.append(z.imag / TINY)
    f = ends[0] - ends[1]
    J = torch.stack((ders[0][0], ders[0][1], -ders[1][0], -ders[1][1], ders[0][2] - ders[1][2]), dim=-1)
    r, g = (f * f).sum(1), 2.0 * (f[:, :, None] * J).sum(1)
    if case["mode"] == "adjoint":
        return {"r": r, "grad": g[:, :4].contiguous(), "grad_e": g[:, 4].sum()}
    return {"f": f, "r": r, "grad": g, "J": J}


def _triangles(grid):
    """Corners (n_tris, 3, 4) in the order p1, p2, p3 of Sec. 6.2.4 and the
    (theta, s) of each corner."""
    v, theta, s, periodic = grid
    th, sv = _dev(theta), _dev(s)
    if periodic:
        v, th = torch.cat((v, v[:, :1]), dim=1), torch.cat((th, th[:1] + TWO_PI))
    full = torch.cat((v, th[None, :, None].expand(*v.shape[:2], 1), sv[:, None, None].expand(*v.shape[:2], 1)), dim=-1)
    a, b, c, d = full[:-1, :-1], full[:-1, 1:], full[1:, :-1], full[1:, 1:]     # W(i,k) W(i+1,k) W(i,k+1) W(i+1,k+1)
    t = torch.stack((torch.stack((b, a, c), dim=2), torch.stack((c, d, b), dim=2)), dim=2)
    return t.reshape(-1, 3, 6), (full.shape[0] - 1, full.shape[1] - 1)


def _overlaps(la, ha, lb, hb, i, j):
    return ((la[i] <= hb[j]) & (lb[j] <= ha[i])).all(1)


def _box_pairs(ta, qa, tb, qb):
    """Pairs of triangles whose closed boxes overlap, by halving blocks of
    quads (each block's box is the box of its triangles)."""
    levels = []
    for t, (ms_, nt) in ((ta, qa), (tb, qb)):
        lo = t[:, :, :4].amin(1).reshape(ms_, nt, 2, 4).amin(2)
        hi = t[:, :, :4].amax(1).reshape(ms_, nt, 2, 4).amax(2)
        lv = [(lo, hi)]
        while lv[-1][0].shape[0] * lv[-1][0].shape[1] > 1:
            l, h = lv[-1]
            pad = (0, 0, 0, l.shape[1] % 2, 0, l.shape[0] % 2)
            l = torch.nn.functional.pad(l, pad, value=math.inf)
            h = torch.nn.functional.pad(h, pad, value=-math.inf)
            m, n = l.shape[0] // 2, l.shape[1] // 2
            lv.append((l.reshape(m, 2, n, 2, 4).amin((1, 3)), h.reshape(m, 2, n, 2, 4).amax((1, 3))))
        levels.append(lv)
    A, B = levels
    ka, kb = len(A) - 1, len(B) - 1
    i = j = torch.zeros(1, dtype=torch.int64, device="cuda")

    def children(lv, k, i):
        (m, n), (mp, np_) = lv[k - 1][0].shape[:2], lv[k][0].shape[:2]
        r, c = 2 * (i // np_), 2 * (i % np_)
        rr = torch.stack((r, r, r + 1, r + 1), dim=1)
        cc = torch.stack((c, c + 1, c, c + 1), dim=1)
        return rr * n + cc, (rr < m) & (cc < n)

    while ka or kb:
        if ka >= kb:
            ch, ok = children(A, ka, i)
            i, j, ka = ch[ok], j[:, None].expand(-1, 4)[ok], ka - 1
        else:
            ch, ok = children(B, kb, j)
            i, j, kb = i[:, None].expand(-1, 4)[ok], ch[ok], kb - 1
        (la, ha), (lb, hb) = ((x.reshape(-1, 4) for x in lv[k]) for lv, k in ((A, ka), (B, kb)))
        keep = _overlaps(la, ha, lb, hb, i, j)
        i, j = i[keep], j[keep]
    i = (2 * i[:, None] + torch.tensor([0, 0, 1, 1], device="cuda")).reshape(-1)
    j = (2 * j[:, None] + torch.tensor([0, 1, 0, 1], device="cuda")).reshape(-1)
    la, ha, lb, hb = (f(1) for t in (ta, tb) for f in (t[:, :, :4].amin, t[:, :, :4].amax))
    keep = _overlaps(la, ha, lb, hb, i, j)
    return i[keep], j[keep]


def _exact_hits(a, b):
    """(values (n_hits, 13), hits ordered by triangle numbers) of a mesh pair."""
    ta, qa = _triangles(a)
    tb, qb = _triangles(b)
    i, j = _box_pairs(ta, qa, tb, qb)
    P, Q = ta[i], tb[j]
    M = torch.stack((P[:, 0, :4] - P[:, 1, :4], P[:, 2, :4] - P[:, 1, :4], Q[:, 1, :4] - Q[:, 0, :4],
                     Q[:, 1, :4] - Q[:, 2, :4]), dim=-1)
    z, info = torch.linalg.solve_ex(M, (Q[:, 1, :4] - P[:, 1, :4])[..., None])
    z = z[..., 0]
    u, v, p, q = z.unbind(1)
    ins = (info == 0) & (z >= 0).all(1) & (u + v <= 1) & (p + q <= 1)
    u, v, p, q, P, Q, i, j = (x[ins] for x in (u, v, p, q, P, Q, i, j))
    at = lambda T, x, y: T[:, 1] + x[:, None] * (T[:, 0] - T[:, 1]) + y[:, None] * (T[:, 2] - T[:, 1])  # noqa: E731
    fa, fb = at(P, u, v), at(Q, p, q)
    margin = torch.stack((u, v, p, q, 1 - (u + v), 1 - (p + q)), dim=1).amin(1) if len(u) else u
    out = torch.cat((torch.stack((u, v, p, q), dim=1), fa[:, :4],
                     torch.stack((_wrap(a, fa[:, 4]), fa[:, 5], _wrap(b, fb[:, 4]), fb[:, 5], margin), dim=1)), dim=1)
    return out[torch.argsort(i * tb.shape[0] + j)]


def _wrap(grid, theta):
    return torch.where(theta >= TWO_PI, theta - TWO_PI, theta) if grid[3] else theta


def _exact_search(case, seed):
    if case["kind"] == "pair":
        rows = [_exact_hits(*pair) for pair in _pair_grids(case, seed)]
    elif case["kind"] == "batch":
        rows = [_exact_hits(*pair) for pair in _batch_grids(case, seed)]
    else:
        (u, th_u, s_u, _), (s, th_s, s_s, _) = _layer_grids(case, seed)

        def half(v, th, sv, layer, sign):
            b0, b1 = sorted((sign * DOM * LAM ** (layer - 1), sign * DOM * LAM ** layer))
            k0, k1 = int(np.argmin(np.abs(sv - b0))), int(np.argmin(np.abs(sv - b1)))
            return v[k0:k1 + 1], th, sv[k0:k1 + 1], True

        rows = [_exact_hits(half(u, th_u, s_u, n, a), half(s, th_s, s_s, m, b))
                for n in range(1, case["n_layers"] + 1) for a in (1, -1) for m in (n, n - 1) for b in (1, -1)]
    hits = torch.cat(rows)
    values = torch.zeros((max(HITS_CAP[case["kind"]], len(hits)), 13), dtype=torch.float64, device="cuda")
    values[:len(hits)] = hits
    return {"values": values}       # the rest is whole numbers


def exact(case, seed):
    kind = case["kind"]
    if kind == "patches":
        return None             # millions of candidates and no hits to speak of: its counts say what it does
    if kind in HITS_CAP:
        return _exact_search(case, seed)
    if kind == "map":
        f, mu = (_field_puls, MU_PULS) if case["frame"] == "pulsating" else (_field_pm, MU_PM)
        return _gbs(f, _states(case, seed).T.contiguous(), case["periods"], mu, ECC).T.contiguous()
    if kind == "matrix":
        y = _states(case, seed)
        eye = torch.eye(4, dtype=torch.float64, device="cuda")
        out, cols = _flow_jet(_field_pm, y, [eye[c].expand_as(y) for c in range(4)], case["periods"], MU_PM, ECC)
        return out, torch.stack(cols, dim=-1)
    if kind == "shift":
        rho = _dev(np.random.default_rng(seed).uniform(-math.pi, math.pi, case["rows"]))
        return _shifted(_rows(case, seed), rho, case["order"])
    if kind == "interp":
        rng = np.random.default_rng(seed)
        at = torch.tensor(rng.integers(0, case["rows"], case["queries"]), device="cuda")
        return _interpolated(_rows(case, seed), at, _dev(rng.uniform(0, TWO_PI, case["queries"])))
    if kind == "chart":
        return _exact_chart(case, seed)
    return _exact_refine(case, seed)
