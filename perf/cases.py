"""Measured cases of the framework: what a Newton-type simulator has it do,
through the public entry points of ``paper_2411_06224_amd``.

Inputs are made on the GPU with plain torch from the seed alone:

* ``cube``: an n^3 grid of unit cells, five tetrahedra each, nodes displaced by
  uniform noise, linear elastic element matrices plus lumped mass
  (``H = M + h^2 sum K_e``), and stiff contact couplings between surface
  nodes; the framework's own benchmark runs the 48^3 cube (117,649 nodes, 9.0
  million listed blocks, 20,000 contacts), its tests the 1^3 to 8^3 cubes.
* ``sheet``: a triangle sheet with in-plane stiffness, bending pairs and
  affine bodies lying on it, with vertex-face and edge-edge contact blocks;
  the benchmark runs 512^2 cells with 2,000 bodies, the tests 64^2.

Solves run to a tight residual (1e-10), so that the solution is determined by
the system and not by the iteration at which the recurrence stops; a solve to
1e-4 is the same launches, fewer times.
"""

import math

import numpy as np
import torch

import paper_2411_06224_amd as mp

_DEV = "cuda"
_DT = 0.01  # time step of H = M + dt^2 K


def listed():
    return [
        # one matrix-vector product of the smallest tested system: launch latency
        {"name": "spmv_8_f64", "kind": "spmv", "n": 8, "dtype": "f64"},
        # the same of the benchmark's system: matrix streaming
        {"name": "spmv_48_f64", "kind": "spmv", "n": 48, "dtype": "f64"},
        # FP32 values on a size that is no multiple of anything
        {"name": "spmv_31_f32", "kind": "spmv", "n": 31, "dtype": "f32"},
        # the preconditioner inside a caller's own Krylov method, mixed precision
        {"name": "apply_21_mixed", "kind": "apply", "n": 21, "precision": "mixed"},
        # the numeric phase of every Newton step and the first use of its result
        {"name": "build_48_f64", "kind": "build", "n": 48, "precision": "f64"},
        # the smallest solve: latency and launches
        {"name": "solve_8_f64", "kind": "solve", "n": 8, "E": 1e5, "precision": "f64"},
        # an ordinary solve in mixed precision, odd size
        {"name": "solve_33_mixed", "kind": "solve", "n": 33, "E": 1e6, "precision": "mixed"},
        # the benchmark's system: build and solve of one Newton step
        {"name": "solve_48_f64", "kind": "solve", "n": 48, "E": 1e6, "precision": "f64"},
        # differentiable solve, forward and backward, gradients of H and b
        {"name": "grad_16_f64", "kind": "grad", "n": 16, "E": 1e6},
        # assembly of every element and contact block of the benchmark's system
        {"name": "assemble_48", "kind": "assemble", "n": 48, "noalloc": False},
        # assembly of a small system without device allocation
        {"name": "assemble_9_noalloc", "kind": "assemble", "n": 9, "noalloc": True},
        # a whole Newton step's linear algebra with changed contacts: contact
        # reduction, assembly, re-plan, build and solve
        {"name": "newton_256", "kind": "newton", "cells": 256, "bodies": 500, "contacts": 60000},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["spmv", "apply", "build", "solve", "solve", "grad", "assemble", "newton"])
    if kind == "spmv":
        return {"kind": kind, "n": size(4, 48), "dtype": rng.choice(["f64", "f32"])}
    if kind in ("apply", "build"):
        return {"kind": kind, "n": size(4, 48), "precision": rng.choice(["f64", "mixed"])}
    if kind == "solve":
        return {"kind": kind, "n": size(4, 40), "E": 10.0 ** rng.randint(5, 7),
                "precision": rng.choice(["f64", "mixed"])}
    if kind == "grad":
        return {"kind": kind, "n": size(4, 28), "E": 10.0 ** rng.randint(5, 6)}
    if kind == "assemble":
        noalloc = rng.random() < 0.5
        return {"kind": kind, "n": size(4, 26 if noalloc else 48), "noalloc": noalloc}
    cells = size(48, 224)
    return {"kind": kind, "cells": cells, "bodies": max(4, cells * cells // rng.randint(120, 260)),
            "contacts": max(100, int(cells * cells * rng.uniform(0.3, 0.9)))}


# ------------------------------------------------------------------- inputs


def _generator(seed, salt):
    g = torch.Generator(device=_DEV)
    g.manual_seed(1000003 * (int(seed) % (1 << 40)) + salt)
    return g


def _uniform(g, *shape):
    return torch.rand(*shape, generator=g, device=_DEV, dtype=torch.float64)


def _cross(a, b):
    return torch.stack([a[:, 1] * b[:, 2] - a[:, 2] * b[:, 1], a[:, 2] * b[:, 0] - a[:, 0] * b[:, 2],
                        a[:, 0] * b[:, 1] - a[:, 1] * b[:, 0]], 1)


def _cube_mesh(n):
    """Node grid positions [V, 3] (cell units) and tetrahedra [T, 4]."""
    m = n + 1
    ar = torch.arange(m, device=_DEV)
    k, j, i = torch.meshgrid(ar, ar, ar, indexing="ij")
    grid = torch.stack([i.reshape(-1), j.reshape(-1), k.reshape(-1)], 1).to(torch.float64)
    ac = torch.arange(n, device=_DEV)
    k, j, i = (t.reshape(-1) for t in torch.meshgrid(ac, ac, ac, indexing="ij"))
    corner = torch.stack([(i + (c & 1)) + m * ((j + ((c >> 1) & 1)) + m * (k + (c >> 2))) for c in range(8)], 1)
    even = torch.tensor([[0, 3, 5, 6], [1, 0, 3, 5], [2, 0, 3, 6], [4, 0, 5, 6], [7, 3, 5, 6]], device=_DEV)
    odd = torch.tensor([[1, 2, 4, 7], [0, 1, 2, 4], [3, 1, 2, 7], [5, 1, 4, 7], [6, 2, 4, 7]], device=_DEV)
    par = ((i + j + k) % 2 == 1)[:, None, None]
    pick = torch.where(par, odd[None], even[None]).reshape(-1, 20)
    return grid, torch.gather(corner, 1, pick).reshape(-1, 4)


def _pairs(nodes):
    """(rows, cols) of all pairs of each row of nodes [k, w]."""
    w = nodes.shape[1]
    a = torch.arange(w, device=_DEV).repeat_interleave(w)
    b = torch.arange(w, device=_DEV).repeat(w)
    return nodes[:, a].reshape(-1), nodes[:, b].reshape(-1)


def _rank_one(weight, normal, k):
    """Blocks k w_a w_b n n^T of every pair of the w weights."""
    ww = (weight[:, :, None] * weight[:, None, :]).reshape(weight.shape[0], -1)
    nn = normal[:, :, None] * normal[:, None, :]
    return ((k[:, None] * ww)[:, :, None, None] * nn[:, None]).reshape(-1, 3, 3)


def _stiff(g, n, w):
    """Listed 3x3 blocks of n contact matrices Q diag(s) Q^T of 3w rows, Q a
    product of reflections, s log-uniform in [1e2, 1e6]."""
    d = 3 * w
    Q = torch.eye(d, device=_DEV, dtype=torch.float64).expand(n, d, d)
    for _ in range(3):
        v = torch.randn(n, d, generator=g, device=_DEV, dtype=torch.float64)
        v = v / v.norm(dim=1, keepdim=True)
        Q = Q - 2 * (Q * v[:, None, :]).sum(-1)[:, :, None] * v[:, None, :]
    s = torch.exp(math.log(1e2) + math.log(1e4) * _uniform(g, n, d))
    M = torch.zeros(n, d, d, device=_DEV, dtype=torch.float64)
    for k in range(d):
        M += (s[:, k, None] * Q[:, :, k])[:, :, None] * Q[:, None, :, k]
    M = 0.5 * (M + M.transpose(1, 2))
    return M.reshape(n, w, 3, w, 3).permute(0, 1, 3, 2, 4).reshape(-1, 3, 3)


def _cube_blocks(n, E, seed, nu=0.45, rho=1000.0):
    """Listed blocks (rows, cols, blocks) of the cube and the mesh edges."""
    g = _generator(seed, 17)
    h = 0.4 / 8 if n <= 8 else 1.0 / n
    grid, tet = _cube_mesh(n)
    V = grid.shape[0]
    x = h * (grid + 0.1 * (2 * _uniform(g, V, 3) - 1))
    p = x[tet]
    e1, e2, e3 = p[:, 1] - p[:, 0], p[:, 2] - p[:, 0], p[:, 3] - p[:, 0]
    c1, c2, c3 = _cross(e2, e3), _cross(e3, e1), _cross(e1, e2)
    det = (e1 * c1).sum(1, keepdim=True)
    gr = torch.stack([-(c1 + c2 + c3), c1, c2, c3], 1) / det[:, :, None]
    vol = det[:, 0].abs() / 6
    lam, mu = E * nu / ((1 + nu) * (1 - 2 * nu)), E / (2 * (1 + nu))
    outer = gr[:, :, None, :, None] * gr[:, None, :, None, :]  # [T, a, b, i, j] = g_a,i g_b,j
    dot = (gr[:, :, None, :] * gr[:, None, :, :]).sum(-1)
    eye = torch.eye(3, device=_DEV, dtype=torch.float64)
    K = lam * outer + mu * outer.transpose(-1, -2) + mu * dot[..., None, None] * eye
    K = (_DT * _DT * vol)[:, None, None, None, None] * K
    rows, cols = _pairs(tet)
    mass = torch.zeros(V, device=_DEV, dtype=torch.float64)
    order = torch.sort(tet.reshape(-1), stable=True)
    _add_sorted(mass, order.values, (rho / 4 * vol).repeat_interleave(4)[order.indices])
    R, C, B = [rows, torch.arange(V, device=_DEV)], [cols, torch.arange(V, device=_DEV)], [
        K.reshape(-1, 3, 3), mass[:, None, None] * eye]
    # contacts: pairs of surface nodes two cells apart along one axis (the
    # same pairs for every seed: a simulator's contacts outlive a Newton step)
    nc = 20000 * n * n // (48 * 48)
    if nc:
        gp = _generator(n, 3)
        on = ((grid == 0) | (grid == n)).any(1)
        surf = torch.nonzero(on)[:, 0]
        a = surf[torch.randint(0, surf.numel(), (4 * nc,), generator=gp, device=_DEV)]
        axis = torch.randint(0, 3, (4 * nc,), generator=gp, device=_DEV)
        to = grid[a].clone()
        to[torch.arange(4 * nc, device=_DEV), axis] += 2
        inside = (to <= n).all(1)
        b = (to[:, 0] + (n + 1) * (to[:, 1] + (n + 1) * to[:, 2])).to(torch.int64)
        ok = inside & on[torch.where(inside, b, 0)]
        a, b = a[ok][:nc], b[ok][:nc]
        r, c = _pairs(torch.stack([a, b], 1))
        R.append(r), C.append(c), B.append(_stiff(g, a.numel(), 2))
    edges = torch.cat([tet[:, [i, j]] for i in range(4) for j in range(i + 1, 4)])
    return V, torch.cat(R), torch.cat(C), torch.cat(B), edges


def _add_sorted(out, index, value):
    """out[index] += value for ascending index, each in the listed order."""
    at, counts = torch.unique_consecutive(index, return_counts=True)
    start = torch.cumsum(counts, 0) - counts
    for k in range(int(counts.max()) if counts.numel() else 0):
        sel = torch.nonzero(counts > k)[:, 0]
        out[at[sel]] += value[start[sel] + k]


def _sum_blocks(V, rows, cols, blocks):
    """3x3-block CSR (row_ptr, col_idx, val) of listed blocks, equal ones
    summed in list order."""
    key, order = torch.sort(rows * V + cols, stable=True)
    uniq, seg = torch.unique_consecutive(key, return_inverse=True)
    val = torch.zeros(uniq.numel(), 3, 3, device=_DEV, dtype=torch.float64)
    _add_sorted(val, seg, blocks[order])
    row_ptr = torch.searchsorted(uniq, torch.arange(V + 1, device=_DEV) * V)
    return row_ptr.to(torch.int32), (uniq % V).to(torch.int32), val


def _graph(V, edges):
    """Host CSR of the undirected node graph."""
    key = torch.unique(torch.cat([edges[:, 0] * V + edges[:, 1], edges[:, 1] * V + edges[:, 0]]))
    ptr = torch.searchsorted(key, torch.arange(V + 1, device=_DEV) * V)
    return ptr.to(torch.int32).cpu().numpy(), (key % V).to(torch.int32).cpu().numpy()


def _normal(seed, salt, n):
    return torch.randn(n, generator=_generator(seed, salt), device=_DEV, dtype=torch.float64)


def _cube_system(case, seed):
    V, r, c, blk, edges = _cube_blocks(case["n"], case.get("E", 1e6), seed)
    rp, ci, val = _sum_blocks(V, r, c, blk)
    return V, rp, ci, val, edges


def _sheet_system(case, seed, dt=_DT, side=0.05):
    """The sheet with bodies: listed blocks of the system without contacts,
    contact nodes and listed contact blocks."""
    cells, nb, nc = case["cells"], case["bodies"], case["contacts"]
    g = _generator(seed, 29)
    m, h = cells + 1, 1.0 / cells
    Vs = m * m
    ar = torch.arange(cells, device=_DEV)
    j, i = (t.reshape(-1) for t in torch.meshgrid(ar, ar, indexing="ij"))
    a, b, c, d = i + m * j, i + 1 + m * j, i + m * (j + 1), i + 1 + m * (j + 1)
    tri = torch.cat([torch.stack([a, b, d], 1), torch.stack([a, d, c], 1)])
    nt = tri.shape[0]
    area = torch.full((nt,), 0.5 * h * h, device=_DEV, dtype=torch.float64)
    # in-plane stiffness, diagonal blocks along the material axes
    pos = h * torch.stack([torch.arange(Vs, device=_DEV) % m, torch.arange(Vs, device=_DEV) // m], 1).to(torch.float64)
    p = pos[tri]
    gx = torch.stack([p[:, 1, 1] - p[:, 2, 1], p[:, 2, 1] - p[:, 0, 1], p[:, 0, 1] - p[:, 1, 1]], 1) / (2 * area)[:, None]
    gy = torch.stack([p[:, 2, 0] - p[:, 1, 0], p[:, 0, 0] - p[:, 2, 0], p[:, 1, 0] - p[:, 0, 0]], 1) / (2 * area)[:, None]
    s = 0.08 * _uniform(g, nt, 2)
    w = (dt * dt * 5e6 * 1e-3) * area
    kx = (w * (1 + s[:, 0]))[:, None, None] * gx[:, :, None] * gx[:, None, :]
    ky = (w * (1 + s[:, 1]))[:, None, None] * gy[:, :, None] * gy[:, None, :]
    kz = (w * 0.1)[:, None, None] * (gx[:, :, None] * gx[:, None, :] + gy[:, :, None] * gy[:, None, :])
    K = torch.diag_embed(torch.stack([kx, ky, kz], -1)).reshape(-1, 3, 3)
    R, C = _pairs(tri)
    R, C, B = [R], [C], [K]
    # bending: one pair of opposite nodes per interior diagonal
    quad = torch.stack([b, c, a, d], 1)
    wt = torch.tensor([1.0, 1.0, -1.0, -1.0], device=_DEV, dtype=torch.float64).expand(quad.shape[0], 4)
    up = torch.tensor([0.0, 0.0, 1.0], device=_DEV, dtype=torch.float64).expand(quad.shape[0], 3)
    r, c2 = _pairs(quad)
    R.append(r), C.append(c2), B.append(_rank_one(wt, up, (dt * dt * 1e-3 / (h * h)) * (1 + _uniform(g, quad.shape[0]))))
    eye = torch.eye(3, device=_DEV, dtype=torch.float64)
    ids = torch.arange(Vs, device=_DEV)
    R.append(ids), C.append(ids), B.append((200.0 * 1e-3 * h * h) * eye.expand(Vs, 3, 3))
    # bodies: reduced mass and the orthogonality stiffness of A near I
    half = 0.5 * side
    corner = torch.tensor([[sx, sy, sz] for sx in (-half, half) for sy in (-half, half) for sz in (-half, half)],
                          device=_DEV, dtype=torch.float64)
    vol = side ** 3
    J = torch.cat([torch.ones(8, 1, device=_DEV, dtype=torch.float64), corner], 1)
    M4 = (1000.0 * vol / 8) * (J[:, :, None] * J[:, None, :]).sum(0)
    Hb = (M4[:, :, None, None] * eye).expand(nb, 4, 4, 3, 3).clone()
    A = eye + 1e-3 * torch.randn(nb, 3, 3, generator=g, device=_DEV, dtype=torch.float64)  # columns A_k = A[:, k]
    ko = dt * dt * 4e8 * vol
    for x in range(3):
        for y in range(x, 3):
            # gradient of A_x . A_y: A_y in column x and A_x in column y
            v = torch.zeros(nb, 3, 3, device=_DEV, dtype=torch.float64)
            v[:, x] += A[:, y]
            v[:, y] += A[:, x]
            f = v.reshape(nb, 9)
            o = (ko * (1.0 if x == y else 2.0)) * (f[:, :, None] * f[:, None, :])
            Hb[:, 1:, 1:] += o.reshape(nb, 3, 3, 3, 3).permute(0, 1, 3, 2, 4)
    base = Vs + 4 * torch.arange(nb, device=_DEV)
    r, c2 = _pairs(base[:, None] + torch.arange(4, device=_DEV))
    R.append(r), C.append(c2), B.append(Hb.reshape(-1, 3, 3))
    # each body holds on to 16 sheet nodes anywhere (the same for every seed)
    gp = _generator(cells, 7)
    held = torch.randint(0, Vs, (nb, 16), generator=gp, device=_DEV).reshape(-1, 1)
    r, c2 = _pairs(torch.cat([(base[:, None] + torch.arange(4, device=_DEV)).repeat_interleave(16, 0), held], 1))
    R.append(r), C.append(c2), B.append(_stiff(g, 16 * nb, 5))
    V = Vs + 4 * nb
    # contact nodes: sheet nodes and the bodies' corners
    node_row = torch.cat([ids, base.repeat_interleave(8)]).to(torch.int32)
    is_body = torch.cat([torch.zeros(Vs, device=_DEV), torch.ones(8 * nb, device=_DEV)]).to(torch.int32)
    xbar = torch.cat([torch.zeros(Vs, 3, device=_DEV, dtype=torch.float64), corner.repeat(nb, 1)])
    # where the bodies lie and touch: the same for every seed, too
    centre = torch.randint(2, cells - 2, (nb, 2), generator=gp, device=_DEV)
    nvf = nc * 5 // 6
    bd = torch.randint(0, nb, (nvf,), generator=gp, device=_DEV)
    kc = 2 * torch.randint(0, 4, (nvf,), generator=gp, device=_DEV)
    ci = centre[bd] + torch.randint(-1, 1, (nvf, 2), generator=gp, device=_DEV)
    t = ci[:, 0] + cells * ci[:, 1] + cells * cells * torch.randint(0, 2, (nvf,), generator=gp, device=_DEV)
    vf = torch.cat([(Vs + 8 * bd + kc)[:, None], tri[t]], 1)
    nee = nc - nvf
    order = torch.argsort(centre[:, 0] * (4 * cells) + centre[:, 1], stable=True)
    at = torch.randint(0, nb - 1, (nee,), generator=gp, device=_DEV)
    k1 = torch.randint(0, 8, (nee,), generator=gp, device=_DEV)
    k2 = torch.randint(0, 8, (nee,), generator=gp, device=_DEV)
    ee = torch.stack([Vs + 8 * order[at] + k1, Vs + 8 * order[at] + (k1 + 1) % 8, Vs + 8 * order[at + 1] + k2,
                      Vs + 8 * order[at + 1] + (k2 + 3) % 8], 1)
    cr, cc = _pairs(torch.cat([vf, ee]))
    con = (cr.to(torch.int32), cc.to(torch.int32), _stiff(g, nc, 4))
    edges = torch.cat([tri[:, [0, 1]], tri[:, [1, 2]], tri[:, [2, 0]], torch.stack([b, c], 1)]
                      + [torch.stack([base + x, base + y], 1) for x in range(4) for y in range(x + 1, 4)])
    return V, (torch.cat(R), torch.cat(C), torch.cat(B)), (node_row, is_body, xbar), con, edges


# --------------------------------------------------------------- the cases


def prepare(case, seed):
    kind = case["kind"]
    if kind == "newton":
        V, own, nodes, con, edges = _sheet_system(case, seed)
        rp, ci, _ = _sum_blocks(V, own[0], own[1], own[2])
        solver = mp.MasPcg(rp.cpu().numpy(), ci.cpu().numpy(), graph=_graph(V, edges))
        return {"kind": kind, "V": V, "own_r": own[0].to(torch.int32), "own_c": own[1].to(torch.int32),
                "own_b": own[2], "nodes": nodes, "con": con, "solver": solver, "b": _normal(seed, 5, 3 * V)}
    if kind == "assemble":
        V, r, c, blk, _ = _cube_blocks(case["n"], 1e6, seed)
        s = {"kind": kind, "V": V, "rows": r.to(torch.int32), "cols": c.to(torch.int32), "blocks": blk}
        if case["noalloc"]:
            cap = 40 * V
            s["out"] = (torch.empty(V + 1, dtype=torch.int32, device=_DEV),
                        torch.empty(cap, dtype=torch.int32, device=_DEV),
                        torch.empty(cap, 3, 3, dtype=torch.float64, device=_DEV))
        else:
            s["capacity"] = 16 * V
        return s
    V, rp, ci, val, edges = _cube_system(case, seed)
    b = _normal(seed, 5, 3 * V)
    if kind == "spmv":
        return {"kind": kind, "H": mp.BlockMatrix(rp, ci, val.to(torch.float32) if case["dtype"] == "f32" else val),
                "x": b}
    solver = mp.MasPcg(rp.cpu().numpy(), ci.cpu().numpy(), graph=_graph(V, edges),
                       precision=case.get("precision", "f64"))
    H = mp.BlockMatrix(rp, ci, val)
    s = {"kind": kind, "H": H, "b": b, "solver": solver}
    if kind in ("apply", "build"):
        solver.build(H)  # places the plans; a Newton loop builds again on new values
    if kind == "grad":
        s["w"] = _normal(seed, 6, 3 * V)
    return s


def run(state):
    kind = state["kind"]
    if kind == "spmv":
        return mp.bcsr_spmv(state["H"], state["x"])
    if kind == "apply":
        return state["solver"].apply(state["b"])
    if kind == "build":
        state["solver"].build(state["H"])
        return state["solver"].apply(state["b"])
    if kind == "solve":
        state["solver"].build(state["H"])
        x, _ = state["solver"].solve(state["H"], state["b"], tol=1e-10)
        return x
    if kind == "grad":
        H = state["H"]
        val = H.val.detach().requires_grad_(True)
        b = state["b"].detach().requires_grad_(True)
        x = mp.mas_pcg_solve(state["solver"], mp.BlockMatrix(H.row_ptr, H.col_idx, val), b, tol=1e-10)
        gval, gb = torch.autograd.grad((x * state["w"]).sum(), (val, b))
        return {"x": x.detach(), "dval": gval, "db": gb}
    if kind == "assemble":
        if "out" in state:
            rp, ci, val = state["out"]
            nb = mp.bcsr_assemble_noalloc(state["V"], state["rows"], state["cols"], state["blocks"], rp, ci, val)
            return {"row_ptr": rp, "col_idx": ci[:nb], "val": val[:nb]}
        H = mp.bcsr_assemble(state["V"], state["rows"], state["cols"], state["blocks"], capacity=state["capacity"])
        return {"row_ptr": H.row_ptr, "col_idx": H.col_idx, "val": H.val}
    node_row, is_body, xbar = state["nodes"]
    r, c, blk = mp.abd_contact_blocks(node_row.numel(), node_row, is_body, xbar, *state["con"])
    H = mp.bcsr_assemble(state["V"], torch.cat([state["own_r"], r]), torch.cat([state["own_c"], c]),
                         torch.cat([state["own_b"], blk]), capacity=32 * state["V"])
    solver = state["solver"]
    solver.replan(H.row_ptr, H.col_idx)
    solver.build(H)
    x, _ = solver.solve(H, state["b"], tol=1e-10)
    return {"x": x, "row_ptr": H.row_ptr, "col_idx": H.col_idx, "val": H.val}


def _cube_counts(n):
    """Nodes, stored blocks and listed blocks of a cube (stored: about 13 a node)."""
    V, T = (n + 1) ** 3, 5 * n ** 3
    edges = 3 * n * (n + 1) ** 2 + 3 * n * n * (n + 1)
    contacts = 20000 * n * n // (48 * 48)
    return V, V + 2 * edges + 2 * contacts, 16 * T + V + 4 * contacts


def work(case):
    """Inputs read once and outputs written once (a solve's iterations are
    its own affair); floating operations of one product with each."""
    kind = case["kind"]
    if kind == "newton":
        Vs, nb, nc = (case["cells"] + 1) ** 2, case["bodies"], case["contacts"]
        own = 18 * case["cells"] ** 2 + 16 * case["cells"] ** 2 + Vs + 416 * nb
        V = Vs + 4 * nb
        out = 11 * V
        return {"bytes": 80.0 * (own + 16 * nc) + 76.0 * out + 52.0 * V, "flops": 18.0 * (own + 16 * nc + out)}
    V, nnzb, listed_blocks = _cube_counts(case["n"])
    if kind == "assemble":
        return {"bytes": 80.0 * listed_blocks + 76.0 * nnzb + 4.0 * (V + 1), "flops": 9.0 * listed_blocks}
    val = 36.0 if case.get("dtype") == "f32" else 72.0
    matrix = (val + 4) * nnzb + 4.0 * (V + 1)
    if kind == "spmv":
        return {"bytes": matrix + 48.0 * V, "flops": 18.0 * nnzb}
    parts = -(-V // 16)
    inverse = parts * (48 * 48 * 4 if case.get("precision") == "mixed" else 1176 * 8)
    if kind == "apply":
        return {"bytes": inverse + 48.0 * V, "flops": 2.0 * 2304 * parts}
    invert = 2.0 * 48 ** 3 * parts
    if kind == "build":
        return {"bytes": matrix + 2.0 * inverse + 48.0 * V, "flops": invert + 9.0 * nnzb}
    if kind == "solve":
        return {"bytes": matrix + 2.0 * inverse + 48.0 * V, "flops": invert + 18.0 * nnzb}
    return {"bytes": 2 * matrix + 72.0 * nnzb + 2.0 * inverse + 120.0 * V, "flops": invert + 45.0 * nnzb}


# -------------------------------------------------- the same in plain torch


def _product(V, rp, ci, val):
    """x -> H x for 3x3-block CSR, rows padded to equal length."""
    rp, ci = rp.to(torch.int64), ci.to(torch.int64)
    length = rp[1:] - rp[:-1]
    row = torch.repeat_interleave(torch.arange(V, device=_DEV), length)
    val = val.to(torch.float64)

    def of(x):
        prod = (val * x.reshape(-1, 3)[ci][:, None, :]).sum(-1)
        return torch.zeros(V, 3, device=_DEV, dtype=torch.float64).index_add_(0, row, prod).reshape(-1)

    diag = torch.zeros(V, 3, 3, device=_DEV, dtype=torch.float64)
    diag[row[row == ci]] = val[row == ci]
    return of, diag


def _inverse3(A):
    a, b, c = A[:, 0], A[:, 1], A[:, 2]
    cof = torch.stack([_cross(b, c), _cross(c, a), _cross(a, b)], -1)
    return cof / (a * _cross(b, c)).sum(1)[:, None, None]


def _solved(V, rp, ci, val, b, tol=3e-14):
    """H^-1 b by block-Jacobi conjugate gradients, restarted on the residual."""
    of, diag = _product(V, rp, ci, val)
    Di = _inverse3(diag)

    def prec(r):
        return (Di * r.reshape(-1, 3)[:, None, :]).sum(-1).reshape(-1)

    x = torch.zeros_like(b)
    nb = float(b.norm())
    for _ in range(3):
        r = b - of(x)
        if float(r.norm()) <= tol * nb:
            break
        z = prec(r)
        p, rz = z.clone(), torch.dot(r, z)
        for k in range(20000):
            q = of(p)
            alpha = rz / torch.dot(p, q)
            x = x + alpha * p
            r = r - alpha * q
            if k % 50 == 49 and float(r.norm()) <= 0.3 * tol * nb:
                break
            z = prec(r)
            new = torch.dot(r, z)
            p = z + (new / rz) * p
            rz = new
    return x


def _contact_pairs_exact(nodes, con):
    """DOF blocks of the contact list (every listed block mapped)."""
    node_row, is_body, xbar = nodes
    r, c, blk = con[0].to(torch.int64), con[1].to(torch.int64), con[2]
    w = torch.cat([torch.ones(xbar.shape[0], 1, device=_DEV, dtype=torch.float64), xbar], 1)
    R, C, B = [], [], []
    for x in range(4):
        for y in range(4):
            sel = ((is_body[r] > 0) | (x == 0)) & ((is_body[c] > 0) | (y == 0))
            R.append(node_row[r[sel]].to(torch.int64) + x)
            C.append(node_row[c[sel]].to(torch.int64) + y)
            B.append((w[r[sel], x] * w[c[sel], y])[:, None, None] * blk[sel])
    return torch.cat(R), torch.cat(C), torch.cat(B)


def _summed(V, r, c, blk):
    key = r.to(torch.int64) * V + c.to(torch.int64)
    uniq, seg = torch.unique(key, return_inverse=True)
    val = torch.zeros(uniq.numel(), 3, 3, device=_DEV, dtype=torch.float64).index_add_(0, seg, blk)
    rp = torch.searchsorted(uniq, torch.arange(V + 1, device=_DEV) * V)
    return rp, uniq % V, val


def exact(case, seed):
    kind = case["kind"]
    if kind in ("apply", "build"):
        return None  # defined by the framework's own partition and hierarchy
    if kind == "assemble":
        V, r, c, blk, _ = _cube_blocks(case["n"], 1e6, seed)
        return {"row_ptr": None, "col_idx": None, "val": _summed(V, r, c, blk)[2]}
    if kind == "newton":
        V, own, nodes, con, _ = _sheet_system(case, seed)
        r, c, blk = _contact_pairs_exact(nodes, con)
        rp, ci, val = _summed(V, torch.cat([own[0], r]), torch.cat([own[1], c]), torch.cat([own[2], blk]))
        return {"x": _solved(V, rp, ci, val, _normal(seed, 5, 3 * V)), "row_ptr": None, "col_idx": None, "val": val}
    V, rp, ci, val, _ = _cube_system(case, seed)
    b = _normal(seed, 5, 3 * V)
    if kind == "spmv":
        of, _ = _product(V, rp, ci, val.to(torch.float32) if case["dtype"] == "f32" else val)
        return of(b)
    x = _solved(V, rp, ci, val, b)
    if kind == "solve":
        return x
    lam = _solved(V, rp, ci, val, _normal(seed, 6, 3 * V))
    row = torch.repeat_interleave(torch.arange(V, device=_DEV), (rp[1:] - rp[:-1]).to(torch.int64))
    dval = -lam.reshape(-1, 3)[row][:, :, None] * x.reshape(-1, 3)[ci.to(torch.int64)][:, None, :]
    return {"x": x, "dval": dval, "db": lam}
