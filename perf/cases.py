"""The work that a user of the solver has it do, as cases for timing.

A case is one call, or one short fixed sequence of calls, of the public entry
points of paper_2512_12151_amd.bfal on a stack of Kuhn-split boxes in contact:
`blocks` boxes of nx x ny x nz cells along z, each shifted sideways against
the one below, with point-triangle and edge-edge constraints across every
interface.  Kinds (what a pass is):

  step        the state of the current Newton iterate set from device arrays
              and one Newton step (bf_set_state, bf_newton_step)
  restep      the same after an active-set change (bf_set_constraints too)
  subproblem  Algorithm 2 (bf_solve_subproblem) from a given state and set
  collide     the collision side of an outer iteration: bf_update_active_set,
              then bf_max_step_size, along x -> x_hat
  time_step   Algorithm 1 (bf_time_step) of two colliding blocks, the second
              step of a throw, which carries contacts and friction
  new_mesh    a mesh that arrives in host memory: bf_problem_create, state,
              constraints, one step, the result back on the host
  serve       requests of mixed sizes given to a running server at once, each
              result taken as it is done (host data by nature)
"""
import functools
import math
import time

import numpy as np
import torch

from paper_2512_12151_amd import bfal

DEV = "cuda:0"
PERMS = ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0))
NH, SNH, COR = 0, 1, 2

# what every case holds unless it says otherwise
DEFAULTS = dict(kind="step", blocks=2, nx=4, ny=4, nz=4, n_pt=25, n_ee=40, material="nh", squeeze=1.0, jitter=0.01,
                lam_max=1e3, kappa=1e4, tol=1e-5, precision="fp32", mu_f=0.0, check_every=1, poll_every=16, requests=0)


def listed():
    return [
        # the smallest scene of the tests and the smoke check: two 4^3-cell cubes, 65 contacts; launches and latency
        dict(name="step_tiny", kind="step"),
        # an odd-sized interactive scene: ragged rows, a last slice that is not full, three materials, friction held
        # from the step's start
        dict(name="step_odd", kind="step", blocks=3, nx=11, ny=9, nz=7, n_pt=700, n_ee=900, material="mixed", mu_f=0.2),
        # the precision workload's size (about 120k tets, 12k + 8k constraints) at its tolerance, FP32 blocks
        dict(name="step_mid", kind="step", blocks=5, nx=16, ny=16, nz=16, n_pt=12000, n_ee=8000),
        # the same with BF16 blocks inside the refinement to 1e-6
        dict(name="step_mid_bf16", kind="step", blocks=5, nx=16, ny=16, nz=16, n_pt=12000, n_ee=8000, tol=0.3,
             precision="bf16"),
        # the headline workload: 2.25M tets, 1.0M constraints, blocks compressed by 40 %, PCG to 1e-5
        dict(name="step_large", kind="step", blocks=5, nx=50, ny=50, nz=30, n_pt=600000, n_ee=400000, squeeze=0.6,
             lam_max=1e4, kappa=1e5, check_every=4, poll_every=64),
        # the same mesh late in a time step, near its solution, at the paper's stopping rule of 1e-4, on a set that
        # has just changed: few PCG iterations, so the pattern and the assembly count as they do in a whole simulation
        dict(name="restep_large", kind="restep", blocks=5, nx=50, ny=50, nz=30, n_pt=300000, n_ee=200000, jitter=0.002,
             lam_max=10.0, kappa=10.0, tol=1e-4),
        # Algorithm 2 on an ordinary scene: a few Newton steps with line searches and the multiplier update
        dict(name="subproblem_mid", kind="subproblem", blocks=4, nx=17, ny=15, nz=13, n_pt=3000, n_ee=2500,
             jitter=0.01, lam_max=100.0),
        # collision queries of a scene with a large surface (345k tets, 66k surface edges)
        dict(name="collide_large", kind="collide", blocks=3, nx=40, ny=40, nz=12, n_pt=8000, n_ee=5000, jitter=0.004),
        # one time step of the small friction scene: two 8^3-cell cubes (12k tets), hundreds of small solves
        dict(name="time_step", kind="time_step", nx=8, ny=8, nz=8, n_pt=0, n_ee=0, mu_f=0.5),
        # a mesh new to the program, from host memory to the result in host memory
        dict(name="new_mesh", kind="new_mesh", blocks=2, nx=20, ny=20, nz=20, n_pt=1400, n_ee=900),
        # the serving stream: requests of 2.6k to 81k tets, all at once, on a running server
        dict(name="serve", kind="serve", requests=24, nx=19, ny=19, nz=19, n_pt=0, n_ee=0),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "step", "step", "restep", "subproblem", "collide", "time_step", "new_mesh", "serve"])
    tol = rng.choice([1e-5, 1e-6])
    c = dict(kind=kind, tol=tol)
    if kind == "time_step":
        n = rng.randint(3, 7)
        c.update(nx=n, ny=rng.randint(3, 7), nz=n, n_pt=0, n_ee=0, mu_f=rng.choice([0.0, 0.3, 0.5]), tol=1e-5)
        return c
    if kind == "serve":
        n = rng.randint(8, 17)
        c.update(requests=rng.randint(3, 20), nx=n, ny=n, nz=n, n_pt=0, n_ee=0, tol=1e-5)
        return c
    top = {"step": 36, "restep": 44, "subproblem": 13, "collide": 40, "new_mesh": 24}[kind]
    c.update(blocks=rng.randint(2, 5), nx=log_int(3, top), ny=log_int(3, top), nz=log_int(3, min(top, 24)))
    per = c["nx"] * c["ny"] * (c["blocks"] - 1)
    c.update(n_pt=int(per * rng.uniform(0.5, 4.0)), n_ee=int(per * rng.uniform(0.5, 4.0)), jitter=0.004,
             lam_max=rng.choice([10.0, 100.0, 1000.0]))
    if kind in ("step", "restep", "new_mesh"):
        c["material"] = rng.choice(["nh", "nh", "snh", "cor", "mixed"])
    if kind in ("step", "restep"):
        c["mu_f"] = rng.choice([0.0, 0.0, 0.2])
        if rng.random() < 0.2:
            c.update(precision="bf16", tol=0.3, mu_f=0.0)
    return c


def full(case):
    return {**DEFAULTS, **case}


# ------------------------------------------------------------------ inputs

@functools.lru_cache(maxsize=4)
def mesh(blocks, nx, ny, nz):
    """Cell counts -> (integer node coordinates [N, 3] with the block number, tets [T, 4]), x fastest."""
    mx, my, mz = nx + 1, ny + 1, nz + 1
    k, j, i = torch.meshgrid(torch.arange(mz, device=DEV), torch.arange(my, device=DEV), torch.arange(mx, device=DEV),
                             indexing="ij")
    ijk = torch.stack([i, j, k], -1).reshape(-1, 3)
    ck, cj, ci = torch.meshgrid(torch.arange(nz, device=DEV), torch.arange(ny, device=DEV),
                                torch.arange(nx, device=DEV), indexing="ij")
    corner = torch.stack([ci, cj, ck], -1).reshape(-1, 1, 3)
    steps = torch.zeros(6, 4, 3, dtype=torch.long)
    for p, perm in enumerate(PERMS):
        for a, ax in enumerate(perm):
            steps[p, a + 1] = steps[p, a]
            steps[p, a + 1, ax] += 1
        e = (steps[p, 1:] - steps[p, :1]).double()
        if torch.linalg.det(e) < 0:   # positive orientation
            steps[p, [2, 3]] = steps[p, [3, 2]]
    v = corner[:, None] + steps.to(DEV)[None]
    idx = v[..., 0] + mx * (v[..., 1] + my * v[..., 2])
    nb = mx * my * mz
    tets = torch.cat([idx.reshape(-1, 4) + b * nb for b in range(blocks)]).int()
    return torch.cat([torch.cat([ijk, torch.full_like(ijk[:, :1], b)], 1) for b in range(blocks)]), tets


def face_edges(n1, n2, fam):
    """Vertex (i, j) pairs of one family of a grid face's edges: along x, along y, or the cells' diagonals."""
    di, dj = ((1, 0), (0, 1), (1, 1))[fam]
    j, i = torch.meshgrid(torch.arange(n2 + 1 - dj, device=DEV), torch.arange(n1 + 1 - di, device=DEV), indexing="ij")
    return torch.stack([i.reshape(-1), j.reshape(-1)], 1), (di, dj)


@functools.lru_cache(maxsize=4)
def contacts(blocks, nx, ny, nz, n_pt, n_ee):
    """Constraint rows across the interfaces: the same few neighbours of every vertex and edge, nearest first."""
    mx, nb = nx + 1, (nx + 1) * (ny + 1) * (nz + 1)

    def vid(ij, b, top):
        return ij[:, 0] + mx * ij[:, 1] + (nz * (nx + 1) * (ny + 1) if top else 0) + b * nb

    def inside(ij):
        return (ij[:, 0] >= 0) & (ij[:, 0] <= nx) & (ij[:, 1] >= 0) & (ij[:, 1] <= ny)

    ring = sorted(((di, dj) for di in range(-4, 4) for dj in range(-4, 4)),
                  key=lambda o: ((o[0] + 0.5) ** 2 + (o[1] + 0.5) ** 2, o))
    j, i = torch.meshgrid(torch.arange(ny + 1, device=DEV), torch.arange(nx + 1, device=DEV), indexing="ij")
    p = torch.stack([i.reshape(-1), j.reshape(-1)], 1)
    rows, have = [], 0
    for di, dj in ring:
        for tri in (((0, 0), (1, 0), (1, 1)), ((0, 0), (0, 1), (1, 1))):
            for b in range(blocks - 1):
                for top in (True, False):   # the lower block's top vertices, then the upper block's bottom ones
                    t = [p + torch.tensor([di + a, dj + c], device=DEV) for a, c in tri]
                    ok = inside(t[0]) & inside(t[2])
                    r = torch.stack([vid(p, b if top else b + 1, top)] +
                                    [vid(q, b + 1 if top else b, not top) for q in t], 1)[ok]
                    rows.append(r)
                    have += len(r)
        if have >= n_pt:
            break
    pt = (torch.cat(rows)[:n_pt] if n_pt else torch.zeros(0, 4, device=DEV)).int().contiguous()
    rows, have = [], 0
    for di, dj in ring:
        for fa, fb in ((0, 1), (1, 0), (2, 0), (2, 1), (0, 2), (1, 2)):
            e, (ei, ej) = face_edges(nx, ny, fa)
            gi, gj = ((1, 0), (0, 1), (1, 1))[fb]
            g0 = e + torch.tensor([di, dj], device=DEV)
            g1 = g0 + torch.tensor([gi, gj], device=DEV)
            ok = inside(g0) & inside(g1)
            for b in range(blocks - 1):
                r = torch.stack([vid(e, b, True), vid(e + torch.tensor([ei, ej], device=DEV), b, True),
                                 vid(g0, b + 1, False), vid(g1, b + 1, False)], 1)[ok]
                rows.append(r)
                have += len(r)
        if have >= n_ee:
            break
    ee = (torch.cat(rows)[:n_ee] if n_ee else torch.zeros(0, 4, device=DEV)).int().contiguous()
    return pt, ee


def scene(c, seed):
    """Device arrays of one scene, from the case and the seed alone."""
    g = torch.Generator(device=DEV).manual_seed(1000003 * (seed % (1 << 30)) + 17)

    def uniform(lo, hi, *n):
        return lo + (hi - lo) * torch.rand(*n, generator=g, device=DEV, dtype=torch.float64)

    grid, tets = mesh(c["blocks"], c["nx"], c["ny"], c["nz"])
    a, gap = 1.0 / max(c["nx"], c["ny"]), 1e-3
    N, T = len(grid), len(tets)
    b = grid[:, 3]
    shift = (uniform(0.1, 0.4, c["blocks"], 2) * a).cumsum(0)   # sideways, against the block below
    rest = grid[:, :3].double() * a
    rest[:, :2] += shift[b]
    rest[:, 2] += b * (c["nz"] * a + gap)
    fixed = ((b == 0) & (grid[:, 2] == 0)) | ((b == c["blocks"] - 1) & (grid[:, 2] == c["nz"]) & (c["squeeze"] < 1.0))
    x = rest.clone()
    x[:, 2] *= c["squeeze"]
    free = (~fixed).double()[:, None]
    x_hat = x + c["jitter"] * a * c["squeeze"] * torch.randn(N, 3, generator=g, device=DEV, dtype=torch.float64) * free
    pt, ee = contacts(c["blocks"], c["nx"], c["ny"], c["nz"], c["n_pt"], c["n_ee"])
    n = len(pt) + len(ee)
    stiff = torch.exp(uniform(math.log(5e4), math.log(2e5), c["blocks"]))
    E = stiff[torch.arange(c["blocks"], device=DEV).repeat_interleave(T // c["blocks"])]
    mat = {"nh": None, "snh": torch.full((T,), SNH), "cor": torch.full((T,), COR),
           "mixed": torch.arange(T) // (6 * c["nx"]) % 3}[c["material"]]
    return dict(tets=tets, rest=rest, E=E, nu=torch.full_like(E, 0.4), rho=torch.full_like(E, 1000.0),
                fixed=fixed.to(torch.uint8), material=None if mat is None else mat.int().to(DEV), x=x, x_hat=x_hat,
                x_tilde=x.clone(), dt=0.01, pt=pt, ee=ee, lam=torch.exp(uniform(0.0, math.log(c["lam_max"]), n)),
                gamma=torch.ones(n, dtype=torch.float64, device=DEV), kappa=c["kappa"], delta=1e-3)


def to_host(sc):
    return {k: v.cpu().numpy() if isinstance(v, torch.Tensor) else v for k, v in sc.items()}


def problem(ctx, sc):
    return bfal.Problem(ctx, sc["tets"], sc["rest"], sc["E"], sc["nu"], sc["rho"], sc["fixed"], sc["material"])


def set_state(pb, sc):
    pb.set_state(sc["x"], sc["x_hat"], sc["x_tilde"], sc["dt"])


def set_constraints(pb, sc):
    pb.set_constraints(sc["pt"], sc["ee"], sc["lam"], sc["gamma"], sc["kappa"], sc["delta"])


def request_case(c, i):
    """Request i of a serving case: two stacked cubes of 6 cells up to the case's, 0.4 contacts per surface vertex."""
    lo, hi = 6, max(6, c["nx"])
    n = int(round(math.exp(math.log(lo) + (math.log(hi) - math.log(lo)) * ((0.5 + i * 0.6180339887) % 1.0))))
    m = int(0.4 * 12 * n * n)
    return {**c, "blocks": 2, "nx": n, "ny": n, "nz": n, "n_pt": 6 * m // 10, "n_ee": m - 6 * m // 10}


def solve_opts(c):
    bf16 = c["precision"] == "bf16"
    return dict(tol=c["tol"], max_iter=20000, precision=bfal.BF_PREC_BF16_REFINE if bf16 else bfal.BF_PREC_FP32,
                check_every=c["check_every"], poll_every=c["poll_every"])


def time_step_kw(c):
    return dict(tol=c["tol"], mu_f=c["mu_f"], eps_v=1e-3, k_min=6 if c["mu_f"] > 0 else 2)


# --------------------------------------------------- the five entry points

def prepare(case, seed):
    c = full(case)
    kind = c["kind"]
    s = dict(case=c)
    if kind == "serve":
        s["requests"] = [to_host(scene(request_case(c, i), seed * 64 + i)) for i in range(c["requests"])]
        s["server"] = bfal.Server(0, max_active=64)
        s["next_id"] = 0
        return s
    s["ctx"] = ctx = bfal.Context(0)
    sc = scene(c, seed)
    if kind == "new_mesh":
        s["scene"] = to_host(sc)
        return s
    if kind == "time_step":
        g = torch.Generator(device=DEV).manual_seed(seed % (1 << 30))
        sc["x"] = sc["x"] + 1e-5 * torch.randn(sc["x"].shape, generator=g, device=DEV, dtype=torch.float64) * (
            sc["fixed"] == 0)[:, None]
        sc["x_hat"] = sc["x"].clone()
        sc["x_tilde"] = sc["x"].clone()
        half = len(sc["x"]) // 2   # the upper block is thrown down and sideways onto the lower one
        sc["x_tilde"][half:] += sc["dt"] * torch.tensor([0.2, 0.0, -0.5], device=DEV, dtype=torch.float64)
        torch.cuda.synchronize()
        pb = problem(ctx, sc)
        set_state(pb, sc)
        set_constraints(pb, sc)
        x, v, _, _ = pb.time_step(**time_step_kw(c))   # the step that lands it
        pt, ee, lam, gam = pb.constraints()
        x1 = torch.from_numpy(x).to(DEV)
        sc.update(x=x1, x_hat=x1.clone(), x_tilde=x1 + sc["dt"] * torch.from_numpy(v).to(DEV),
                  pt=torch.from_numpy(pt).to(DEV), ee=torch.from_numpy(ee).to(DEV), lam=torch.from_numpy(lam).to(DEV),
                  gamma=torch.from_numpy(gam).to(DEV))
        s.update(pb=pb, scene=sc)
        return s
    if kind == "collide":   # block b moves down by 1.4 b gaps into the one below
        grid, _ = mesh(c["blocks"], c["nx"], c["ny"], c["nz"])
        free = (sc["fixed"] == 0).double()
        sc["x_hat"][:, 2] -= 1.4e-3 * grid[:, 3].double() * free
        cap = 3 * (c["n_pt"] + c["n_ee"]) + 16 * (c["nx"] + 1) * (c["ny"] + 1) * (c["blocks"] - 1)
        s["rows"], s["multipliers"] = np.full((cap, 4), -1, np.int32), np.zeros((2, cap))
    torch.cuda.synchronize()
    s["scene"] = sc
    s["pb"] = pb = problem(ctx, sc)
    set_state(pb, sc)
    set_constraints(pb, sc)
    if c["mu_f"] > 0.0:
        pb.set_friction(c["mu_f"], 1e-3)
    s["p"] = torch.empty_like(sc["x"])
    torch.cuda.synchronize()
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "serve":
        server, ids, got = s["server"], {}, [None] * len(s["requests"])
        for i, r in enumerate(s["requests"]):
            server.submit(s["next_id"], r, tol=c["tol"])
            ids[s["next_id"]] = i
            s["next_id"] += 1
        while ids:
            done = server.poll()
            for q in done:
                got[ids.pop(q)] = server.result(q)[0]
            if not done:
                time.sleep(5e-5)
        return got
    sc = s["scene"]
    if kind == "new_mesh":
        pb = problem(s["ctx"], sc)
        set_state(pb, sc)
        set_constraints(pb, sc)
        p, _, _ = pb.newton_step(**solve_opts(c))
        pb.close()
        return p
    pb = s["pb"]
    set_state(pb, sc)
    if kind == "step":
        p, _, _ = pb.newton_step(out=s["p"], **solve_opts(c))
        return p
    set_constraints(pb, sc)
    if kind == "restep":
        p, _, _ = pb.newton_step(out=s["p"], **solve_opts(c))
        return p
    if kind == "subproblem":
        x_hat, lam, gam, st, _ = pb.solve_subproblem(tol=c["tol"], max_newton=8)
        return dict(x_hat=x_hat, lam=lam, gamma=gam, energy=st["energy_final"])
    if kind == "collide":
        pb.update_active_set()
        alpha, _ = pb.max_step_size()
        rows, mult = s["rows"], s["multipliers"]   # the program's own buffers, larger than any set it meets
        pt, ee, lam, gam = pb.constraints()
        n = len(pt) + len(ee)
        rows[: len(pt)], rows[len(pt):n] = pt, ee
        mult[0, :n], mult[1, :n] = lam, gam
        return dict(rows=rows, multipliers=mult, n_pt=len(pt), n_ee=len(ee), alpha=alpha)
    x, v, _, _ = pb.time_step(**time_step_kw(c))
    return dict(x=x, v=v)


def sizes(c):
    """(nodes, tets, stored upper blocks of the merged pattern, constraints), the blocks to a few per cent."""
    N = c["blocks"] * (c["nx"] + 1) * (c["ny"] + 1) * (c["nz"] + 1)
    T = 6 * c["blocks"] * c["nx"] * c["ny"] * c["nz"]
    per = max(1, 2 * (c["blocks"] - 1) * (c["nx"] + 1) * (c["ny"] + 1))
    n = c["n_pt"] + c["n_ee"]
    return N, T, int(7.4 * N) + int(min(4.0 * n, 9.0 * per)), n


def iterations(c):
    """PCG iterations of one solve, roughly: the cells along the longest way through the stack, and the tolerance."""
    if c["kappa"] >= 1e5:
        return 9000
    way = max(c["nx"], c["ny"], c["blocks"] * c["nz"])
    return int(4 * way * (1.0 if c["tol"] < 5e-5 else 0.7)) if c["precision"] == "fp32" else 20 * way


def work(case):
    """Inputs read once and the result written once per assembly, the matrix and four vectors once per iteration."""
    c = full(case)
    if c["kind"] == "serve":
        w = [work({**request_case(c, i), "kind": "new_mesh"}) for i in range(c["requests"])]
        return {k: sum(q[k] for q in w) for k in ("bytes", "flops")}
    N, T, nnzb, n = sizes(c)
    assemble = {"bytes": 40.0 * T + 121.0 * N + 32.0 * n + 40.0 * nnzb, "flops": 2500.0 * T + 400.0 * n}
    solve = {"bytes": 40.0 * nnzb + 48.0 * N, "flops": 36.0 * nnzb + 40.0 * N}
    if c["kind"] == "collide":
        faces = 4 * c["blocks"] * (c["nx"] * c["ny"] + c["nz"] * (c["nx"] + c["ny"]))
        return {"bytes": 16.0 * T + 48.0 * N + 64.0 * n + 200.0 * faces, "flops": 100.0 * T + 30000.0 * faces}
    steps = {"subproblem": 3, "time_step": 8}.get(c["kind"], 1)
    its = iterations(c)
    return {k: steps * (assemble[k] + its * solve[k]) for k in ("bytes", "flops")}


# ------------------------------------------- the Newton step in 64 bits

def closest(X, is_pt):
    """Closest points of point-triangle or edge-edge rows X [n, 4, 3]: distance, normal, weights."""
    def dot(u, v):
        return (u * v).sum(-1)

    def clamp(p, u, e):
        return (dot(p - u, e) / dot(e, e)).clamp(0.0, 1.0)

    n = len(X)
    zero, one = torch.zeros(n, dtype=X.dtype, device=X.device), torch.ones(n, dtype=X.dtype, device=X.device)
    if is_pt:
        p, t = X[:, 0], [X[:, 1], X[:, 2], X[:, 3]]
        e1, e2, r = t[1] - t[0], t[2] - t[0], p - t[0]
        a11, a12, a22, r1, r2 = dot(e1, e1), dot(e1, e2), dot(e2, e2), dot(e1, r), dot(e2, r)
        det = a11 * a22 - a12 * a12
        u, v = (a22 * r1 - a12 * r2) / det, (a11 * r2 - a12 * r1) / det
        cand = [(torch.stack([one, u + v - 1.0, -u, -v], 1), (u >= 0) & (v >= 0) & (u + v <= 1))]
        for k in range(3):
            w = torch.zeros(n, 4, dtype=X.dtype, device=X.device)
            s = clamp(p, t[k], t[(k + 1) % 3] - t[k])
            w[:, 0], w[:, 1 + k], w[:, 1 + (k + 1) % 3] = 1.0, s - 1.0, -s
            cand.append((w, torch.ones_like(one, dtype=torch.bool)))
    else:
        a0, a1, b0, b1 = X.unbind(1)
        ea, eb, r = a1 - a0, b1 - b0, a0 - b0
        aa, bb, ab, ar, br = dot(ea, ea), dot(eb, eb), dot(ea, eb), dot(ea, r), dot(eb, r)
        det = aa * bb - ab * ab
        s, t = (-ar * bb + ab * br) / det, (aa * br - ab * ar) / det
        cand = []
        for s_, t_, ok in ((s, t, (s >= 0) & (s <= 1) & (t >= 0) & (t <= 1)), (zero, clamp(a0, b0, eb), None),
                           (one, clamp(a1, b0, eb), None), (clamp(b0, a0, ea), zero, None),
                           (clamp(b1, a0, ea), one, None)):
            cand.append((torch.stack([1.0 - s_, s_, t_ - 1.0, -t_], 1),
                         torch.ones_like(one, dtype=torch.bool) if ok is None else ok))
    W = torch.stack([w for w, _ in cand], 1)
    D = torch.einsum("nca,nak->nck", W, X)
    d = torch.where(torch.stack([ok for _, ok in cand], 1), D.norm(dim=2), math.inf)
    k = d.argmin(1)
    at = torch.arange(n, device=X.device)
    diff, w = D[at, k], W[at, k]
    d = diff.norm(dim=1)
    return d, diff / d[:, None], w


def stress_and_hessian(F, mu, lam, mat):
    """P [T, 3, 3] and d2Psi/dF2 [T, 9, 9] of every tet's material, by directional derivatives of P."""
    eye = torch.eye(3, dtype=F.dtype, device=F.device)
    J, Fi = torch.linalg.det(F), torch.linalg.inv(F)
    FiT, lnJ = Fi.transpose(1, 2), torch.log(J)
    U, S, Vh = torch.linalg.svd(F)
    R = U @ Vh
    Sy = R.transpose(1, 2) @ F
    tr = Sy.diagonal(dim1=1, dim2=2).sum(1)
    solve = torch.linalg.inv(tr[:, None, None] * eye - Sy)
    mu_, lam_, J_, lnJ_, tr_ = (v[:, None, None] for v in (mu, lam, J, lnJ, tr))
    code = mat[:, None, None]
    P = torch.where(code == NH, mu_ * (F - FiT) + lam_ * lnJ_ * FiT,
                    torch.where(code == SNH, mu_ * F + (lam_ * (J_ - 1.0) - mu_) * J_ * FiT,
                                2.0 * mu_ * (F - R) + lam_ * (tr_ - 3.0) * R))
    cols = []
    for q in range(9):
        dF = torch.zeros_like(F)
        dF[:, q // 3, q % 3] = 1.0
        A = FiT @ dF.transpose(1, 2) @ FiT   # -d(F^-T)
        t = (Fi * dF.transpose(1, 2)).sum((1, 2))[:, None, None]
        K = R.transpose(1, 2) @ dF
        ax = torch.stack([K[:, 2, 1] - K[:, 1, 2], K[:, 0, 2] - K[:, 2, 0], K[:, 1, 0] - K[:, 0, 1]], 1)
        o = (solve @ ax[:, :, None])[:, :, 0]
        z = torch.zeros_like(o[:, 0])
        Om = torch.stack([z, -o[:, 2], o[:, 1], o[:, 2], z, -o[:, 0], -o[:, 1], o[:, 0], z], 1).reshape(-1, 3, 3)
        dR = R @ Om
        dtr = (R * dF).sum((1, 2))[:, None, None]
        d_nh = mu_ * dF + (mu_ - lam_ * lnJ_) * A + lam_ * t * FiT
        d_snh = mu_ * dF + lam_ * J_ * t * J_ * FiT + (lam_ * (J_ - 1.0) - mu_) * J_ * (t * FiT - A)
        d_cor = 2.0 * mu_ * (dF - dR) + lam_ * dtr * R + lam_ * (tr_ - 3.0) * dR
        cols.append(torch.where(code == NH, d_nh, torch.where(code == SNH, d_snh, d_cor)).reshape(-1, 9))
    return P, torch.stack(cols, 2)


def newton_exact(sc, mu_f):
    """p = -H^-1 G in 64 bits from plain torch and numpy: assembled as a sparse matrix, solved by a dense
    factorization up to 9000 unknowns and by block-Jacobi CG to 1e-13 above."""
    N, tets, x, xh = len(sc["x"]), sc["tets"].long(), sc["x"], sc["x_hat"]
    X = sc["rest"][tets]
    Dm = (X[:, 1:] - X[:, :1]).transpose(1, 2)
    Di = torch.linalg.inv(Dm)
    vol = torch.linalg.det(Dm).abs() / 6.0
    mu, lam = sc["E"] / (2 * (1 + sc["nu"])), sc["E"] * sc["nu"] / ((1 + sc["nu"]) * (1 - 2 * sc["nu"]))
    Y = xh[tets]
    F = (Y[:, 1:] - Y[:, :1]).transpose(1, 2) @ Di
    mat = sc["material"] if sc["material"] is not None else torch.zeros(len(tets), dtype=torch.int32, device=DEV)
    P, H9 = stress_and_hessian(F, mu, lam, mat)
    A = torch.cat([-Di.sum(1, keepdim=True), Di], 1)   # rows A_a
    w, Q = np.linalg.eigh(H9.add(H9.transpose(1, 2)).mul(0.5).cpu().numpy())
    w, Q = torch.from_numpy(np.maximum(w, 0.0)).to(DEV), torch.from_numpy(Q).to(DEV)
    hv = sc["dt"] ** 2 * vol
    Bm = torch.einsum("taj,ik->tijak", A, torch.eye(3, dtype=A.dtype, device=DEV)).reshape(-1, 9, 12)
    half = (Q * w.sqrt()[:, None, :]).transpose(1, 2).contiguous() @ Bm
    blocks = [(tets, hv[:, None, None] * (half.transpose(1, 2).contiguous() @ half))]
    mass = torch.zeros(N, dtype=torch.float64, device=DEV).index_add_(
        0, tets.reshape(-1), (sc["rho"] * vol / 4.0).repeat_interleave(4))
    G = mass[:, None] * (xh - sc["x_tilde"])
    G.index_add_(0, tets.reshape(-1), torch.einsum("t,tij,taj->tai", hv, P, A).reshape(-1, 3))
    ids = torch.cat([sc["pt"], sc["ee"]]).long()
    if len(ids):
        parts = [closest(x[r.long()], k == 0) for k, r in enumerate((sc["pt"], sc["ee"])) if len(r)]
        d, nrm, wt = (torch.cat(v) for v in zip(*parts))
        cv = d + torch.einsum("na,nak,nk->n", wt, xh[ids] - x[ids], nrm) - sc["delta"]
        k, lm, gm = sc["kappa"], sc["lam"], sc["gamma"]
        gf = k * gm * (cv - lm / k - (cv - lm / k).clamp(min=0.0))
        grad = (wt[:, :, None] * nrm[:, None, :]).reshape(-1, 12)
        G.index_add_(0, ids.reshape(-1), (gf[:, None] * grad).reshape(-1, 3))
        blocks.append((ids, (k * gm)[:, None, None] * grad[:, :, None] * grad[:, None, :]))
        if mu_f > 0.0:
            e, coef = 1e-3 * sc["dt"], mu_f * (lm - k * (d - sc["delta"])).clamp(min=0.0)
            v = torch.einsum("na,nak->nk", wt, xh[ids] - x[ids])
            Pn = torch.eye(3, dtype=torch.float64, device=DEV) - nrm[:, :, None] * nrm[:, None, :]
            u = (Pn @ v[:, :, None])[:, :, 0]
            y = u.norm(dim=1)
            t = u / torch.where(y > 0, y, 1.0)[:, None]
            f1y = torch.where(y >= e, 1.0 / torch.where(y > 0, y, 1.0), 2.0 / e - y / e ** 2)
            f1p = torch.where(y >= e, 0.0, 2.0 / e - 2.0 * y / e ** 2)
            K = coef[:, None, None] * (f1y[:, None, None] * Pn + (f1p - f1y)[:, None, None] * t[:, :, None] * t[:, None])
            G.index_add_(0, ids.reshape(-1), (wt[:, :, None] * ((coef * f1y)[:, None] * u)[:, None]).reshape(-1, 3))
            blocks.append((ids, (wt[:, :, None, None, None] * wt[:, None, None, :, None] * K[:, None, :, None, :]
                                 ).reshape(-1, 12, 12)))
    free = (sc["fixed"] == 0).double().repeat_interleave(3)
    rows, cols, vals = [torch.arange(3 * N, device=DEV)] * 2 + [mass.repeat_interleave(3)]
    rows, cols, vals = [rows], [cols], [vals]
    for q, v in blocks:
        dof = (3 * q[:, :, None] + torch.arange(3, device=DEV)).reshape(-1, 12)
        rows.append(dof.repeat_interleave(12, 1).reshape(-1))
        cols.append(dof.repeat(1, 12).reshape(-1))
        vals.append(v.reshape(-1))
    rows, cols, vals = torch.cat(rows), torch.cat(cols), torch.cat(vals)
    vals = torch.where(rows == cols, vals, vals * free[rows] * free[cols])
    H = torch.sparse_coo_tensor(torch.stack([rows, cols]), vals, (3 * N, 3 * N)).coalesce()
    b = -(G.reshape(-1) * free)
    if 3 * N <= 9000:
        return torch.from_numpy(np.linalg.solve(H.to_dense().cpu().numpy(), b.cpu().numpy())).reshape(N, 3)
    i, v = H.indices(), H.values()
    D = torch.zeros(N, 3, 3, dtype=torch.float64, device=DEV)
    same = i[0] // 3 == i[1] // 3
    D[i[0][same] // 3, i[0][same] % 3, i[1][same] % 3] = v[same]
    D, H = torch.linalg.inv(D), H.to_sparse_csr()
    p, r = torch.zeros_like(b), b.clone()
    z = (D @ r.reshape(N, 3, 1)).reshape(-1)
    q, rz, stop = z.clone(), r @ z, 1e-13 * b.norm()
    for it in range(30000):
        h = H @ q
        al = rz / (q @ h)
        p += al * q
        r -= al * h
        z = (D @ r.reshape(N, 3, 1)).reshape(-1)
        new = r @ z
        q = z + (new / rz) * q
        rz = new
        if it % 32 == 31 and r.norm() <= stop:
            break
    return p.reshape(N, 3)


def exact(case, seed):
    """The exact direction of a Newton step; the other kinds stop by rules of their own (a line search, a conservative
    collision time, a termination weight) and have no such value."""
    c = full(case)
    if c["kind"] == "serve":
        cs = [request_case(c, i) for i in range(c["requests"])]
        return [newton_exact(scene(q, seed * 64 + i), 0.0) if i < 6 else None for i, q in enumerate(cs)]
    if c["kind"] not in ("step", "restep", "new_mesh") or sizes(c)[1] > 130000:
        return None
    return newton_exact(scene(c, seed), c["mu_f"])
