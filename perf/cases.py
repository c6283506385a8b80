"""Performance cases: the work a user has this library do, through its public
entry points (`paper_1708_00744_amd.dsu`).

`listed()` names the cases, `draw(rng)` gives one more of the same ranges,
`prepare(case, seed)` builds what a user's program holds before the call,
`run(state)` is one pass, `work(case)` the bytes and operations a pass cannot
do without, and `exact(case, seed)` the outputs of a first pass in 64 bits,
computed with plain numpy and torch.

Inputs.  Electrons sit near the sites of a cubic lattice (0.3 spacings of
uniform jitter): like an equilibrated Metropolis configuration, and unlike
independent uniform points, that keeps electrons apart, so the Slater matrices
are as well conditioned as a running simulation's.  Orbitals are plane waves in
a box of side 10.  The mixed FP32 form's numbers are handed on in float32, the
precision its ratios are computed in; everything else in float64.
"""
import numpy as np
import torch

from paper_1708_00744_amd import dsu

L = 10.0
FORMS = {"fp64": dsu.FP64, "fp32": dsu.FP32_MIXED}
TWIST = np.array([0.31, -0.17, 0.42])  # boundary twist of the complex orbitals
SETS = 3                               # proposals held for consecutive host-driven passes


# ------------------------------------------------------------------- cases
def listed():
    return [
        # Host-driven moves, one propose and one accept or reject call each.
        # A small molecule: every launch and wait shows.  sigma = 0.05 L gives
        # an acceptance near 0.65, so rejections take part.  With "inverse" the
        # pass ends in a measurement: the host reads A^-1 for its estimators.
        {"name": "walker_n64_k16", "kind": "walker", "form": "fp64", "n": 64, "k": 16, "moves": 64, "sigma": 0.5,
         "inverse": True},
        # The mid-size FP64 walker of the delay study, at high acceptance.
        {"name": "walker_n1024_k64", "kind": "walker", "form": "fp64", "n": 1024, "k": 64, "moves": 256,
         "sigma": 0.002},
        # The largest host-driven walker: mixed FP32, orbital rows already on the device, deep window.
        {"name": "walker_fp32_n4096_k128", "kind": "walker", "form": "fp32", "n": 4096, "k": 128, "moves": 256,
         "sigma": 0.002},
        # Drift-diffusion (DMC) moves: the drift at the present point, ratio and gradient at the proposed one.
        {"name": "drift_n1000_k32", "kind": "drift", "form": "fp64", "n": 1000, "k": 32, "moves": 128, "sigma": 0.04},
        # Complex orbitals under a boundary twist, FP64 complex, ragged size.
        {"name": "complex_n500_k16", "kind": "complex", "form": "fp64", "n": 500, "k": 16, "moves": 200,
         "sigma": 0.02, "inverse": True},
        # Moves of a single-reference multideterminant expansion (reference, singles, doubles).
        {"name": "multidet_n1024_k64", "kind": "multidet", "form": "fp64", "n": 1024, "k": 64, "moves": 256,
         "sigma": 0.002, "virt": 16},
        # Direct calculations: a fresh inverse of one complex matrix, and of a
        # population of real ones (the periodic recompute).
        {"name": "inverse_complex_n600", "kind": "inverse", "form": "fp64", "n": 600, "complex": True},
        {"name": "recompute_n1024_w64", "kind": "recompute", "form": "fp64", "n": 1024, "walkers": 64, "spins": 1},
        # Whole Metropolis sweeps on the device.  Many small walkers, mixed FP32, acceptance near 0.99,
        # with the residual watchdog of a production run.
        {"name": "batch_fp32_n512_w512_k32", "kind": "batch", "form": "fp32", "n": 512, "walkers": 512, "spins": 1,
         "k": 32, "sigma": 0.0015, "all": False},
        # Plain FP64, two spins, ragged size, acceptance near 0.5.
        {"name": "batch_fp64_n1000_w16_k64", "kind": "batch", "form": "fp64", "n": 1000, "walkers": 16, "spins": 2,
         "k": 64, "sigma": 0.45, "all": False},
        # The largest population: mixed FP32 at 100 % acceptance, the
        # paper's test regime, with the periodic recompute.
        {"name": "batch_fp32_n4096_w32_k128", "kind": "batch", "form": "fp32", "n": 4096, "walkers": 32, "spins": 1,
         "k": 128, "sigma": 0.0015, "all": True},
        # Serving: a saturated pool of walkers of mixed size, two spins each.
        {"name": "serve_24_requests", "kind": "serve", "form": "fp32", "k": 64, "requests": 24, "sizes":
         "128,256,512,1024,2048", "sweeps": 5, "sigma": 0.05},
    ]


def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return min(hi, max(lo, round(lo * (hi / lo) ** rng.random())))


def draw(rng):
    kind = rng.choice(["walker", "walker", "drift", "complex", "multidet", "inverse", "recompute", "batch", "batch",
                       "batch", "serve"])
    sigma = round(10.0 ** rng.uniform(-2.8, -0.4), 5)
    if kind == "walker":
        form = rng.choice(["fp64", "fp32"])
        n = _log(rng, 48, 2048 if form == "fp64" else 4096)
        return {"kind": kind, "form": form, "n": n, "k": min(n, _log(rng, 1, 128)),
                "moves": min(n, rng.randint(48, 256)), "sigma": sigma, "inverse": n <= 600 and rng.random() < 0.5}
    if kind in ("drift", "complex", "multidet"):
        n = _log(rng, 48, {"drift": 2048, "complex": 1100, "multidet": 1500}[kind])
        if kind != "complex":  # short time steps
            sigma = min(sigma, 0.04)
        case = {"kind": kind, "form": "fp64", "n": n, "k": min(n, _log(rng, 1, 64)),
                "moves": min(n, rng.randint(40, 160)), "sigma": sigma, "inverse": n <= 600 and rng.random() < 0.5}
        return dict(case, virt=rng.randint(3, 24)) if kind == "multidet" else case
    if kind == "inverse":
        cplx = rng.random() < 0.5
        return {"kind": kind, "form": "fp64", "n": _log(rng, 64, 900 if cplx else 2048), "complex": cplx}
    if kind == "recompute":
        n = _log(rng, 100, 2048)
        return {"kind": kind, "form": rng.choice(["fp64", "fp32"]), "n": n, "spins": 1,
                "walkers": max(1, min(256, int(rng.uniform(0.1, 1.0) * 2.0**26 / n**2)))}
    if kind == "batch":
        # a mixed FP32 walker with a deep window runs at 100 % acceptance
        # (where deep windows pay), the others by Metropolis
        form, k = rng.choice(["fp64", "fp32"]), _log(rng, 8, 128)
        n, spins = _log(rng, 100, 1500 if form == "fp64" else 3000), rng.choice([1, 2])
        every = form == "fp32" and k > 64
        return {"kind": kind, "form": form, "n": n, "walkers": max(1, min(256, int(2.0**25.5 / n**2 / spins))),
                "spins": spins, "k": min(k, n), "sigma": 0.0015 if every else sigma, "all": every}
    sizes = sorted({_log(rng, 100, 1500) for _ in range(3)})
    return {"kind": "serve", "form": "fp32", "k": rng.choice([32, 64]), "requests": rng.randint(6, 16),
            "sizes": ",".join(map(str, sizes)), "sweeps": rng.randint(2, 5), "sigma": sigma}


# ------------------------------------------------------------------ inputs
def _rng(seed, what):
    return np.random.default_rng([int(seed), what])


def _positions(rng, n):
    side = int(np.ceil(n ** (1 / 3) - 1e-9))
    site = rng.permutation(side**3)[:n]
    grid = np.stack([site // side**2, site // side % side, site % side], 1)
    return (grid + 0.5 + rng.uniform(-0.3, 0.3, (n, 3))) * (L / side)


def _vectors(n):
    """(vectors, kind) of the n real plane waves: 1, then cos and sin by shells."""
    r = int((3 * n / (8 * np.pi)) ** (1 / 3) * 2) + 2
    g = np.arange(-r, r + 1)
    v = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    x, y, z = v.T
    v = v[(x > 0) | ((x == 0) & ((y > 0) | ((y == 0) & (z > 0))))]
    v = v[np.lexsort((v[:, 2], v[:, 1], v[:, 0], (v * v).sum(1)))]
    vec = np.concatenate([np.zeros((1, 3), int), np.repeat(v, 2, 0)])[:n]
    kind = np.concatenate([[0], np.tile([1, 2], len(v))])[:n]
    return vec.astype(np.float64), kind


def _phase(pos, vec):
    return 2 * np.pi / L * (pos @ vec.T)


def _rows(pos, vec, kind):
    ph = _phase(pos, vec)
    out = np.cos(ph)
    out[..., kind == 2] = np.sin(ph[..., kind == 2])
    return out


def _grad_rows(pos, vec, kind):
    """(moves, 3, n) derivatives of the rows."""
    ph = _phase(pos, vec)
    d = np.where(kind == 1, -np.sin(ph), np.where(kind == 2, np.cos(ph), 0.0))
    return 2 * np.pi / L * vec.T[None] * d[:, None, :]


def _twisted(n):
    r = int((3 * n / (4 * np.pi)) ** (1 / 3)) + 3
    g = np.arange(-r, r + 1)
    v = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    q = ((v + TWIST) ** 2).sum(1)
    return v[np.lexsort((v[:, 2], v[:, 1], v[:, 0], q))][:n] + TWIST


def _zrows(pos, vec):
    return np.exp(1j * _phase(pos, vec))


def _expansion(n, m):
    """Reference, singles from the highest occupied orbitals, pair doubles; the
    reference dominates, as where a single-reference expansion is used."""
    top = list(range(n - min(8, n), n))
    dets = [(1.0, [])] + [(0.02 / (1 + a + v), [(j, v)]) for a, j in enumerate(top) for v in range(m)]
    dets += [(0.004 / (1 + a + v), [(top[a], v), (top[a + 1], v + 1)]) for a in range(0, len(top) - 1, 2)
             for v in range(0, m - 1, 2)]
    return dets


def _host_inputs(case, seed):
    """Slater matrix, proposals and uniforms of the host-driven kinds: `moves`
    consecutive electrons, SETS proposals each around their first position."""
    n, moves, rng = case["n"], case["moves"], _rng(seed, 1)
    pos = _positions(rng, n)
    prop = [pos[:moves] + case["sigma"] * rng.standard_normal((moves, 3)) for _ in range(SETS)]
    out = {"u": [rng.random(moves) for _ in range(SETS)]}
    if case["kind"] == "complex":
        vec = _twisted(n)
        return dict(out, slater=_zrows(pos, vec), rows=[_zrows(p, vec) for p in prop])
    m = case.get("virt", 0)
    vec, kind = _vectors(n + m)
    full, rows = _rows(pos, vec, kind), [_rows(p, vec, kind) for p in prop]
    out.update(slater=np.ascontiguousarray(full[:, :n]), rows=[np.ascontiguousarray(r[:, :n]) for r in rows])
    if m:
        out.update(virt=np.ascontiguousarray(full[:, n:]), vrows=[np.ascontiguousarray(r[:, n:]) for r in rows],
                   dets=_expansion(n, m))
    if case["kind"] == "drift":
        out.update(grad=_grad_rows(pos[:moves], vec, kind), grads=[_grad_rows(p, vec, kind) for p in prop])
    return out


def _population(case, seed):
    rng = _rng(seed, 2)
    w, s, n = case["walkers"], case["spins"], case["n"]
    pos = np.stack([_positions(rng, n) for _ in range(w * s)]).reshape(w, s, n, 3)
    return pos, rng.integers(1, 2**62, w, dtype=np.int64).astype(np.uint64)


def _requests(case, seed):
    rng = _rng(seed, 3)
    sizes = [int(x) for x in case["sizes"].split(",")]
    out = []
    for i in range(case["requests"]):
        n = sizes[i % len(sizes)]
        out.append({"request_id": i, "n": n, "spins": 2, "seed": int(rng.integers(1, 2**62)), "sigma": case["sigma"],
                    "sweeps": case["sweeps"], "arrival_s": 0.0,
                    "positions": np.stack([_positions(rng, n) for _ in range(2)])})
    return out


def _matrices(case, seed):
    """Two matrices: the walker's own and the one it is given afresh."""
    rng, n = _rng(seed, 4), case["n"]
    pos = [_positions(rng, n) for _ in range(2)]
    if case["complex"]:
        vec = _twisted(n)
        return [_zrows(p, vec) for p in pos]
    vec, kind = _vectors(n)
    return [_rows(p, vec, kind) for p in pos]


# ------------------------------------------------------------------- passes
def prepare(case, seed):
    kind, form = case["kind"], FORMS[case["form"]]
    state = {"case": case, "passes": 0}
    if kind in ("walker", "drift", "multidet"):
        state.update(_host_inputs(case, seed))
        state["walker"] = dsu.Walker(state["slater"], case["k"], precision=form)
        if kind == "multidet":
            state["walker"].set_multidet(state["virt"], state["dets"])
        if form == dsu.FP32_MIXED:  # a program that evaluates its orbitals on the GPU
            state["rows"] = [torch.tensor(r, dtype=torch.float32, device="cuda") for r in state["rows"]]
            torch.cuda.synchronize()
    elif kind == "complex":
        state.update(_host_inputs(case, seed))
        state["walker"] = dsu.ZWalker(state["slater"], case["k"])
    elif kind == "inverse":
        own, state["fresh"] = _matrices(case, seed)
        state["walker"] = dsu.ZWalker(own, 16) if case["complex"] else dsu.Walker(own, 16)
    elif kind in ("recompute", "batch"):
        pos, seeds = _population(case, seed)
        state["batch"] = dsu.Batch(case["n"], pos, seeds, np.arange(len(seeds)), case.get("sigma", 0.1),
                                   case.get("k", 32), precision=form, spins=case["spins"], box_l=L,
                                   recompute_every=20 if form == dsu.FP32_MIXED else 0)
        if kind == "batch" and form == dsu.FP32_MIXED and not case["all"]:
            state["batch"].set_residual_watchdog(16, 1e-2)
    else:
        state["requests"] = _requests(case, seed)
        state["server"] = dsu.Server(case["k"], precision=form, box_l=L, budget_bytes=8 << 30, recompute_every=10)
    return state


def _run_moves(s):
    """One host-driven sweep over the case's electrons; ratios, decisions, log|det|."""
    w, kind, q = s["walker"], s["case"]["kind"], s["passes"] % SETS
    s["passes"] += 1
    rows, us = s["rows"][q], s["u"][q]
    ratio = np.empty(len(us), np.complex128 if kind == "complex" else np.float64)
    taken = np.zeros(len(us), np.int32)
    extra = {}
    if kind == "drift":
        extra = {"drift": np.empty((len(us), 3)), "grad": np.empty((len(us), 3))}
        here, there = s["grad"], s["grads"][q]
    for e in range(len(us)):
        if kind == "drift":
            extra["drift"][e] = w.grad(e, here[e])
            ratio[e], extra["grad"][e] = w.propose_grad(e, rows[e], there[e])
        elif kind == "multidet":
            ratio[e] = w.propose_md(e, rows[e], s["vrows"][q][e])[0]
        elif torch.is_tensor(rows):
            ratio[e] = w.propose_dev(e, rows.data_ptr() + 4 * e * s["case"]["n"])
        else:
            ratio[e] = w.propose(e, rows[e])
        if us[e] < abs(ratio[e]) ** 2:
            w.accept()
            taken[e] = 1
            if kind == "drift":
                here[e] = there[e]
        else:
            w.reject()
    w.flush()
    if s["case"].get("inverse"):
        extra["inverse"] = w.inverse()
    if kind == "complex":
        logabs, phase = w.logdet()
        return dict(extra, ratio=ratio, accepted=taken, logabs=np.float64(logabs), phase=_unit(phase))
    sign, logdet = w.md_value() if kind == "multidet" else w.logdet()
    if s["case"]["form"] == "fp32":
        ratio, extra = ratio.astype(np.float32), {q: x.astype(np.float32) for q, x in extra.items()}
    return dict(extra, ratio=ratio, accepted=taken, sign=sign,
                logdet=np.float32(logdet) if s["case"]["form"] == "fp32" else np.float64(logdet))


def _unit(phase):
    """A phase as a point of the unit circle (no jump at pi)."""
    return np.array([np.cos(phase), np.sin(phase)])


def run(state):
    case = state["case"]
    kind, f32 = case["kind"], case["form"] == "fp32"
    if kind in ("walker", "drift", "multidet", "complex"):
        return _run_moves(state)
    if kind == "inverse":
        # a user that changed the configuration by hand: new matrix in, determinant and inverse out
        w = state["walker"]
        if case["complex"]:
            logabs, phase, _ = w.recompute(state["fresh"])
            return {"logabs": np.float64(logabs), "phase": _unit(phase), "inverse": w.inverse()}
        logdet, sign, _ = w.recompute(state["fresh"])
        return {"logdet": np.float64(logdet), "sign": sign, "inverse": w.inverse()}
    if kind == "serve":
        results, _ = state["server"].run(state["requests"])
        return {"logdet": np.array([r["logdet"] for r in results], np.float32),
                "sign": np.array([r["sign"] for r in results]), "status": np.array([r["status"] for r in results]),
                "accepted": np.array([r["accepted"] for r in results])}
    b = state["batch"]
    if kind == "recompute":
        b.recompute()
    else:
        b.sweep(1, case["all"])
    st = b.stats()
    out = {"logdet": st["logdet"].astype(np.float32) if f32 else st["logdet"], "sign": st["sign"],
           "accepted": st["accepted"], "sweeps": st["sweeps"]}
    if kind == "batch" and not f32:
        out["positions"] = np.stack([b.positions(d) for d in range(b.ndet)])
    return out


# --------------------------------------------------------------------- work
def _move_work(n, k, moves, s, z=1, nx=1, grow=True):
    """Look-ahead moves of one walker: (2 j + 1) rows at j pending moves, and
    the en-bloc update of the inverse after every k.  s: bytes per number, z:
    real products per product (4 if complex), nx: rows proposed per move."""
    bytes_, flops, j = 0.0, 0.0, 0
    for _ in range(moves):
        bytes_ += ((2 * j + 1) + nx) * n * s
        flops += 2.0 * z * n * (nx * (j + 1) + j)
        j += 1
        if j == k:
            bytes_ += 2.0 * n * n * s + 2.0 * k * n * s
            flops += z * (4.0 * n * n * k + 2.0 * n * k * k)
            j = 0
    if j:
        bytes_ += 2.0 * n * n * s + 2.0 * j * n * s
        flops += z * (4.0 * n * n * j + 2.0 * n * j * j)
    return bytes_, flops


def _sweep_work(n, k, s):
    """One sweep of one determinant: a read and a write of its inverse per window."""
    windows = -(-n // k)
    return windows * (2.0 * n * n * s + 2.0 * k * n * s), windows * (4.0 * n * n * k + 2.0 * n * k * k)


def work(case):
    kind, s = case["kind"], 4 if case["form"] == "fp32" else 8
    if kind in ("walker", "multidet", "complex", "drift"):
        n, moves = case["n"], case["moves"]
        z = 4 if kind == "complex" else 1
        b, f = _move_work(n, case["k"], moves, 2 * s if kind == "complex" else s, z, 4 if kind == "drift" else 1)
        if kind == "drift":
            b, f = b + moves * 4.0 * n * s, f + moves * 6.0 * n
        if kind == "multidet":  # the table is read for the proposal and updated on acceptance
            b, f = b + moves * 3.0 * n * case["virt"] * s, f + moves * 4.0 * n * case["virt"]
        return {"bytes": b, "flops": f}
    if kind == "inverse":
        z = 4 if case["complex"] else 1
        n = case["n"]
        return {"bytes": 2.0 * n * n * (16 if case["complex"] else 8), "flops": 2.0 * z * float(n) ** 3}
    if kind == "serve":
        sizes = [int(x) for x in case["sizes"].split(",")]
        b = f = 0.0
        for i in range(case["requests"]):
            n = sizes[i % len(sizes)]
            wb, wf = _sweep_work(n, case["k"], s)
            b, f = b + 2 * (case["sweeps"] * wb + n * n * s), f + 2 * (case["sweeps"] * wf + 2.0 * float(n) ** 3)
        return {"bytes": b, "flops": f}
    n, dets = case["n"], case["walkers"] * case["spins"]
    if kind == "recompute":
        return {"bytes": dets * (24.0 * n + 1.0 * n * n * s), "flops": dets * 2.0 * float(n) ** 3}
    b, f = _sweep_work(n, case["k"], s)
    return {"bytes": dets * b, "flops": dets * f}


# ---------------------------------------------------------- 64-bit reference
def _mulhi(a, b):
    """High 64 bits of the products of uint64 arrays."""
    m = np.uint64(0xFFFFFFFF)
    t = np.uint64(32)
    al, ah, bl, bh = a & m, a >> t, b & m, b >> t
    mid = ah * bl + (al * bl >> t)
    return ah * bh + (mid >> t) + ((mid & m) + al * bh >> t)


def _philox(c, k):
    """Philox4x64-10 blocks of four counter words and two key words (uint64 arrays)."""
    c0, c1, c2, c3 = c
    k0, k1 = k
    m0, m1 = np.uint64(0xD2E7470EE14C6C93), np.uint64(0xCA5A826395121157)
    for _ in range(10):
        c0, c1, c2, c3 = _mulhi(m1, c2) ^ c1 ^ k0, m1 * c2, _mulhi(m0, c0) ^ c3 ^ k1, m0 * c0
        k0, k1 = k0 + np.uint64(0x9E3779B97F4A7C15), k1 + np.uint64(0xBB67AE8584CAA73B)
    return c0, c1, c2, c3


def _draws(seeds, wids, spin, n, sweep):
    """Gaussian steps (w, n, 3) and Metropolis uniforms (w, n) of one sweep."""
    slot = np.uint64(spin * n) + np.arange(n, dtype=np.uint64)[None]
    key = (seeds.astype(np.uint64)[:, None] + 0 * slot, wids.astype(np.uint64)[:, None] + 0 * slot)
    zero, unit = 0 * key[0], lambda x: (x >> np.uint64(11)).astype(np.float64) * 2.0**-53
    with np.errstate(over="ignore"):
        a = _philox((zero + np.uint64(sweep), zero + slot, zero, zero), key)
        b = _philox((zero + np.uint64(sweep), zero + slot, zero + np.uint64(1), zero), key)
    a = [unit(x) for x in a]
    r1, r2 = np.sqrt(-2 * np.log(1 - a[0])), np.sqrt(-2 * np.log(1 - a[2]))
    g = np.stack([r1 * np.cos(2 * np.pi * a[1]), r1 * np.sin(2 * np.pi * a[1]), r2 * np.cos(2 * np.pi * a[3])], -1)
    return g, unit(b[0])


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _t_rows(pos, vec, kind):
    ph = 2 * np.pi / L * (pos @ vec.T)
    return torch.where(kind == 2, torch.sin(ph), torch.cos(ph))


def _metropolis(pos, seeds, wids, spin, sigma, sweeps, every):
    """Sweeps of the walkers' determinants of one spin (w, n, 3) in FP64, each
    accepted move applied at once: positions, log|det|, sign."""
    dev, n = _device(), pos.shape[1]
    vec, kind = (torch.tensor(x, device=dev) for x in _vectors(n))
    p = torch.tensor(pos, device=dev)
    if not every:
        inv = torch.stack([torch.linalg.inv(_t_rows(q, vec, kind)) for q in p])
    for sw in range(sweeps):
        g, u = _draws(seeds, wids, spin, n, sw)
        new = p + sigma * torch.tensor(g, device=dev)
        if every:
            p = new
            continue
        u = torch.tensor(u, device=dev)
        for e in range(n):
            phi = _t_rows(new[:, e], vec, kind)
            t = torch.matmul(phi[:, None, :], inv)[:, 0]
            r = t[:, e].clone()
            ok = (u[:, e] < r * r) & (r.abs() > 1e-12)
            t[:, e] -= 1.0
            t = torch.where(ok[:, None], t / r[:, None], torch.zeros_like(t))
            inv -= inv[:, :, e].clone()[:, :, None] * t[:, None, :]
            p[:, e] = torch.where(ok[:, None], new[:, e], p[:, e])
    ld, sg = [], []
    for w in range(len(p)):
        s, lw = torch.linalg.slogdet(_t_rows(p[w], vec, kind))
        ld.append(float(lw))
        sg.append(int(s))
    return p.cpu().numpy(), np.array(ld), np.array(sg)


def _exact_moves(case, seed):
    """A first host-driven pass with a dense inverse updated at every acceptance."""
    s, dev, kind = _host_inputs(case, seed), _device(), case["kind"]
    a = torch.tensor(s["slater"], device=dev)
    rows = s["rows"][0].astype(np.float32).astype(np.float64) if case["form"] == "fp32" else s["rows"][0]
    rows, us = torch.tensor(rows, device=dev), s["u"][0]
    inv = torch.linalg.inv(a)
    if kind == "drift":
        here, there = (torch.tensor(x, device=dev) for x in (s["grad"], s["grads"][0]))
    if kind == "multidet":
        virt, vrows = torch.tensor(s["virt"], device=dev), torch.tensor(s["vrows"][0], device=dev)
        coef = torch.tensor([c for c, _ in s["dets"]], device=dev)
        occ = torch.zeros((len(coef), 2), dtype=torch.long, device=dev)
        vir = torch.zeros_like(occ)
        order = torch.tensor([len(x) for _, x in s["dets"]], device=dev)
        for d, (_, subs) in enumerate(s["dets"]):
            for q, (j, v) in enumerate(subs):
                occ[d, q], vir[d, q] = j, v

        def psi(table):
            t = [[table[occ[:, x], vir[:, y]] for y in range(2)] for x in range(2)]
            det = torch.where(order == 0, torch.ones_like(coef), torch.where(
                order == 1, t[0][0], t[0][0] * t[1][1] - t[0][1] * t[1][0]))
            return float((coef * det).sum())
        table = torch.matmul(inv, virt)
        value = psi(table)
    ratio, drift, grad = [], [], []
    for e in range(len(us)):
        phi, col = rows[e], inv[:, e].clone()
        t = torch.mv(inv.T, phi)
        r = t[e].item()
        if kind == "drift":
            drift.append(torch.mv(here[e], col).cpu().numpy())
            grad.append(torch.mv(there[e], col).cpu().numpy())
        full = r
        if kind == "multidet":
            x = (vrows[e] - torch.mv(table.T, phi)) / r
            moved = table + col[:, None] * x[None]
            after = psi(moved)
            full = r * after / value
        ratio.append(full)
        if us[e] < abs(full) ** 2:
            t[e] -= 1.0
            inv -= col[:, None] * (t / r)[None]
            a[e] = phi
            if kind == "drift":
                here[e] = there[e]
            if kind == "multidet":
                table, value = moved, after
    sign, logdet = torch.linalg.slogdet(a)
    out = {"ratio": np.array(ratio), "accepted": None}
    if case.get("inverse"):
        out["inverse"] = torch.linalg.inv(a).cpu().numpy()
    if kind == "complex":
        return dict(out, logabs=np.float64(logdet.item()), phase=np.array([sign.real.item(), sign.imag.item()]))
    out.update(sign=None, logdet=np.float64(logdet.item() + (np.log(abs(value)) if kind == "multidet" else 0.0)))
    return dict(out, drift=np.stack(drift), grad=np.stack(grad)) if kind == "drift" else out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("walker", "drift", "multidet", "complex"):
        return _exact_moves(case, seed)
    if kind == "inverse":
        a = torch.tensor(_matrices(case, seed)[1], device=_device())
        sign, logdet = torch.linalg.slogdet(a)
        inv = torch.linalg.inv(a).cpu().numpy()
        if case["complex"]:
            return {"logabs": np.float64(logdet.item()), "phase": np.array([sign.real.item(), sign.imag.item()]),
                    "inverse": inv}
        return {"logdet": np.float64(logdet.item()), "sign": None, "inverse": inv}
    if kind == "serve":
        ld = np.zeros((case["requests"], 2))
        for i, q in enumerate(_requests(case, seed)):
            for s in range(2):
                ld[i, s] = _metropolis(q["positions"][s][None], np.array([q["seed"]]), np.array([i]), s, q["sigma"],
                                       q["sweeps"], False)[1][0]
        return {"logdet": ld, "sign": None, "status": None, "accepted": None}
    pos, seeds = _population(case, seed)
    sweeps = 1 if kind == "batch" else 0
    out = np.zeros((case["walkers"], case["spins"]))
    at = np.zeros_like(pos)
    for s in range(case["spins"]):
        at[:, s], out[:, s], _ = _metropolis(pos[:, s], seeds, np.arange(len(seeds)), s, case.get("sigma", 0.0), sweeps,
                                             case.get("all", True))
    res = {"logdet": out.reshape(-1), "sign": None, "accepted": None, "sweeps": None}
    if kind == "batch" and case["form"] == "fp64":
        res["positions"] = at.reshape(-1, case["n"], 3)
    return res
