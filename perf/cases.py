"""Performance cases of the spectral-element rate: what a solver or a study
built on this package calls, over the sizes, orders, precisions and options it
is called with.

A case is a dict of plain values:

``kind``   the entry point (``volume``, ``ext``, ``affine``, ``surface``,
           ``rhs``, ``autograd``, ``batch``, ``rk3``)
``nq``     nodes per direction; for ``batch`` and ``rk3`` ``orders``, a text of
           several (``"4 6 8 10"``), with ``ne`` elements of each
``ne``     elements; for ``surface`` and ``rhs`` the box ``nx * ny * nz``
``f32``    working precision (FP32, else FP64)
``ref``    perturbation form about the hydrostatic reference state
``acc``    accumulate into the output instead of overwriting it
``nf``     fields of ``ext`` (5, or 8 with the passive tracers)
``rst``    directions of ``ext`` (r+s+t, else the paper's fused r+s)
``walls``  ``surface`` and ``rhs``: boundary faces all round, else periodic

Inputs are seeded synthetic fields of the package's own workloads (warped or
affine hexahedra, a perturbed isentropic atmosphere), made on the GPU.
"""
import math

import numpy as np
import torch

import paper_1604_08501_amd as sv

ATMOSPHERE = (1.0e5, 1.4, 287.0, 9.81)     # p0, gamma, R, gravity
PAPER = (1.0, 1.4, 1.0, 0.0)               # the paper's benchmark kernel
RK_DT = 1.0e-5
LENGTH, WARP = 1000.0, 0.05


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: 64 affine elements of order 4, whose time is the
        # call itself (a unit test, a coarse preconditioner level)
        dict(name="volume_n4_64_f64", kind="volume", nq=5, ne=64, f32=False, ref=True, acc=False),
        # the volume term a full-size solver evaluates per stage: order 7 on
        # 32768 curved elements, FP64
        dict(name="volume_n7_32768_f64", kind="volume", nq=8, ne=32768, f32=False, ref=True,
             acc=False),
        # an odd node count and a ragged element count in FP32, added to terms
        # that were computed before (a partition of a mesh)
        dict(name="volume_n6_5003_f32_acc", kind="volume", nq=7, ne=5003, f32=True, ref=True,
             acc=True),
        # the whole rate v + s of a periodic box, full size, FP64
        dict(name="rhs_n7_32768_f64", kind="rhs", nq=8, nx=32, ny=32, nz=32, f32=False, ref=True,
             acc=False, walls=False),
        # the whole rate of a mid-size box with walls in FP32
        dict(name="rhs_n5_8075_f32_walls", kind="rhs", nq=6, nx=25, ny=19, nz=17, f32=True,
             ref=True, acc=False, walls=True),
        # the surface term added to a volume term computed before
        dict(name="surface_n7_8000_f64_acc", kind="surface", nq=8, nx=20, ny=20, nz=20, f32=False,
             ref=True, acc=True, walls=False),
        # forward and backward of the differentiable volume term
        dict(name="autograd_n7_8192_f64", kind="autograd", nq=8, ne=8192, f32=False, ref=True),
        # the paper's benchmark kernel: r+s, 8 fields, FP32, accumulated
        dict(name="paper_rs_nq8_6912_f32", kind="ext", nq=8, ne=6912, nf=8, rst=False, f32=True,
             ref=False, acc=True),
        # the full volume term with tracers at high order, the same node count
        dict(name="paper_rst_nq12_2048_f32", kind="ext", nq=12, ne=2048, nf=8, rst=True, f32=True,
             ref=False, acc=True),
        # straight-sided meshes: metric terms once per element
        dict(name="affine_n7_32768_f64", kind="affine", nq=8, ne=32768, f32=False, ref=True,
             acc=False),
        # a p-adaptive mesh, four orders in one launch, FP32
        dict(name="batch_n3579_5000_f32", kind="batch", orders="4 6 8 10", ne=5000, f32=True,
             ref=True),
        # one time step of a p-adaptive mesh (three fused stages in a graph)
        dict(name="rk3_n3579_5000_f64", kind="rk3", orders="4 6 8 10", ne=5000, f32=False,
             ref=True),
    ]


def _around(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return max(1, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    kind = rng.choice(["volume", "volume", "rhs", "rhs", "surface", "ext", "ext", "affine",
                       "autograd", "batch", "rk3"])
    f32 = rng.random() < 0.5
    case = dict(kind=kind, f32=f32, ref=rng.random() < 0.8)
    nodes = _around(rng, 2.0e3, 6.0e6)
    if kind in ("batch", "rk3"):
        orders = sorted(rng.sample(range(2, 11), rng.randint(2, 4)))
        nodes = min(nodes, 3000000)
        per = sum(q ** 3 for q in orders)
        case.update(orders=" ".join(str(q) for q in orders), ne=max(1, nodes // per))
        return case
    if kind in ("ext", "affine"):
        nq = rng.choice([4, 5, 6, 7, 8, 9, 10, 12, 16])
    else:
        nq = rng.choice([2, 3, 4, 5, 6, 6, 7, 7, 8, 8, 9, 9, 10, 10])
    case.update(nq=nq)
    ne = max(1, nodes // nq ** 3)
    if kind in ("rhs", "surface"):
        side = ne ** (1.0 / 3.0)
        nx, ny = (max(1, int(round(side * rng.uniform(0.7, 1.4)))) for _ in range(2))
        case.update(nx=nx, ny=ny, nz=max(1, ne // (nx * ny)), walls=rng.random() < 0.4)
    else:
        case.update(ne=ne)
    if kind != "autograd":
        case.update(acc=rng.random() < 0.4)
    if kind == "ext":
        case.update(nf=rng.choice([5, 8]), rst=rng.random() < 0.6)
    return case


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _nodes_and_matrix(nq):
    """Gauss-Lobatto-Legendre nodes and the differentiation matrix, FP64."""
    n = nq - 1
    inner = np.polynomial.legendre.Legendre.basis(n).deriv().roots().real if n > 1 else []
    x = np.concatenate([[-1.0], np.sort(inner), [1.0]])
    x = 0.5 * (x - x[::-1])
    diff = x[:, None] - x[None, :]
    np.fill_diagonal(diff, 1.0)
    w = 1.0 / np.prod(diff, axis=1)
    d = (w[None, :] / w[:, None]) / diff
    np.fill_diagonal(d, 0.0)
    np.fill_diagonal(d, -d.sum(axis=1))
    return x, d


def _pack(a):
    """Cofactors and 1/J of Jacobians a[r][c] (lists of tensors) as 10 slots."""
    slots = []
    for d in range(3):
        for r in range(3):
            r1, r2, d1, d2 = (r + 1) % 3, (r + 2) % 3, (d + 1) % 3, (d + 2) % 3
            slots.append(a[r1][d1] * a[r2][d2] - a[r1][d2] * a[r2][d1])
    jac = a[0][0] * slots[0] + a[1][0] * slots[1] + a[2][0] * slots[2]
    return torch.stack(slots + [1.0 / jac], dim=1)


def _box(case):
    if "nx" in case:
        return case["nx"], case["ny"], case["nz"]
    n = max(1, math.ceil(case["ne"] ** (1.0 / 3.0) - 1e-9))
    return n, n, n


def _warped(nq, ne, box, dev):
    """Metric terms and heights of the first ne elements of a warped box."""
    x1 = torch.from_numpy(_nodes_and_matrix(nq)[0]).to(dev)
    e = torch.arange(ne, device=dev)
    m = torch.arange(nq ** 3, device=dev)
    nx, ny, nz = box
    X = ((e % nx)[:, None] + 0.5 * (x1[m % nq] + 1.0)) / nx
    Y = ((e // nx % ny)[:, None] + 0.5 * (x1[m // nq % nq] + 1.0)) / ny
    Z = ((e // (nx * ny))[:, None] + 0.5 * (x1[m // nq ** 2] + 1.0)) / nz
    pi = math.pi
    sx, cx, sy, cy = torch.sin(pi * X), torch.cos(pi * X), torch.sin(pi * Y), torch.cos(pi * Y)
    sz, cz = torch.sin(pi * Z), torch.cos(pi * Z)
    one = torch.ones_like(X)
    hx, hy, hz = (0.5 * LENGTH / n for n in box)
    wp = WARP * pi
    a = [[one * hx, wp * cy * sz * hy, wp * sy * cz * hz],
         [wp * sz * cx * hx, one * hy, wp * cz * sx * hz],
         [wp * cx * sy * hx, wp * sx * cy * hy, one * hz]]
    return _pack(a), LENGTH * (Z + WARP * sx * sy)


def _affine(nq, ne, box, gen, dev):
    """Per-element metric records of random affine elements, and node heights."""
    x1 = torch.from_numpy(_nodes_and_matrix(nq)[0]).to(dev)
    A = 0.1 * (2.0 * torch.rand(ne, 3, 3, generator=gen, device=dev, dtype=torch.float64) - 1.0)
    A += torch.eye(3, dtype=torch.float64, device=dev)
    m = torch.arange(nq ** 3, device=dev)
    xi = torch.stack([x1[m % nq], x1[m // nq % nq], x1[m // nq ** 2]])
    ez = torch.arange(ne, device=dev) // (box[0] * box[1])
    z = A[:, 2, :] @ xi + (2.0 * ez + 1.0)[:, None]
    return _pack([[A[:, r, c] for c in range(3)] for r in range(3)]), z


def _reference(z):
    """Isentropic hydrostatic rho_ref and Theta_ref at heights z."""
    p0, gamma, r, grav = ATMOSPHERE
    cp, theta0 = gamma * r / (gamma - 1.0), 300.0
    ex = (r * theta0 / p0) ** (gamma - 1.0) - grav * z / (cp * theta0)
    rho = p0 * ex ** (cp / r - 1.0) / (r * theta0)
    return rho, rho * theta0


def _state(ne, nf, nq, gen, dev):
    """rho, momenta, Theta (and tracers) of a perturbed atmosphere."""
    def noise():
        return torch.randn(ne, nq ** 3, generator=gen, device=dev, dtype=torch.float64)
    rho = 1.0 + 0.01 * noise()
    q = [rho, rho * 10.0 * noise(), rho * 10.0 * noise(), rho * 10.0 * noise(),
         rho * (300.0 + noise())]
    q += [rho * (0.2 * i + 0.5 + 0.05 * noise()) for i in range(1, nf - 4)]
    return torch.stack(q, dim=1)


def _neighbours(box, walls, dev):
    """[Ne, 6] elements across r-, r+, s-, s+, t-, t+ (-1 at a wall)."""
    nx, ny, nz = box
    e = torch.arange(nx * ny * nz, device=dev)
    at = [e % nx, e // nx % ny, e // (nx * ny)]
    cols = []
    for d in range(3):
        for step in (-1, 1):
            to = list(at)
            to[d] = (at[d] + step) % box[d]
            n = to[0] + nx * (to[1] + ny * to[2])
            if walls:
                n = torch.where((at[d] + step < 0) | (at[d] + step >= box[d]), -1, n)
            cols.append(n)
    return torch.stack(cols, dim=1).to(torch.int32).contiguous()


def _block(case, nq, ne, box, gen, dev):
    """One order's arrays in the working precision (Theta_ref always FP64)."""
    dt = torch.float32 if case["f32"] else torch.float64
    if case["kind"] == "affine":
        geo, z = _affine(nq, ne, box, gen, dev)
    else:
        geo, z = _warped(nq, ne, box, dev)
    b = dict(D=torch.from_numpy(_nodes_and_matrix(nq)[1]).to(dev, dt), geo=geo.to(dt),
             q=_state(ne, case.get("nf", 5), nq, gen, dev).to(dt), rho_ref=None, theta_ref=None)
    if case["ref"]:
        rho, theta = _reference(z)
        b.update(rho_ref=rho.to(dt), theta_ref=theta.contiguous())
    return b


def _phys(case):
    return PAPER if case["kind"] == "ext" and not case["ref"] else ATMOSPHERE


def _inputs(case, seed):
    """The blocks of the case and what goes with them, made from the seed."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(160408501 + int(seed))
    if "orders" in case:
        box = _box(case)
        return [_block(case, int(t), case["ne"], box, gen, dev) for t in case["orders"].split()]
    box = _box(case)
    ne = case["ne"] if "ne" in case else box[0] * box[1] * box[2]
    b = _block(case, case["nq"], ne, box, gen, dev)
    if case["kind"] in ("rhs", "surface"):
        b["nbr"] = _neighbours(box, case["walls"], dev)
    if case["kind"] == "autograd":
        b["lam"] = torch.randn(b["q"].shape, generator=gen, device=dev, dtype=b["q"].dtype)
    elif case["acc"]:
        b["out"] = torch.randn(b["q"].shape, generator=gen, device=dev, dtype=b["q"].dtype)
    return [b]


def prepare(case, seed):
    blocks = _inputs(case, seed)
    kind, phys = case["kind"], _phys(case)
    if kind == "batch":
        for b in blocks:
            b["rhs"] = torch.empty_like(b["q"])
        return dict(kind=kind, blocks=blocks, plan=sv.BatchPlan(blocks, phys))
    if kind == "rk3":
        q_n = torch.cat([b["q"].reshape(-1) for b in blocks])
        q_1, q_2, rate = (torch.empty_like(q_n) for _ in range(3))
        at = 0
        for b in blocks:
            n, shape = b["q"].numel(), b["q"].shape
            b["q"] = q_n[at:at + n].view(shape)
            b["rhs"] = rate[at:at + n].view(shape)
            at += n
        step = sv.RK3Graph(blocks, q_n, q_1, q_2, rate, RK_DT, phys)
        return dict(kind=kind, blocks=blocks, q_n=q_n, step=step)
    state = dict(blocks[0], kind=kind, phys=phys)
    if kind == "autograd":
        state["q"].requires_grad_(True)
    else:
        state["acc"] = case["acc"]
        state.setdefault("out", torch.empty_like(state["q"]))
    if kind == "ext":
        state["dirs"] = 7 if case["rst"] else 3
    return state


def run(s):
    kind = s["kind"]
    if kind == "batch":
        s["plan"].execute()
        return [b["rhs"] for b in s["blocks"]]
    if kind == "rk3":
        s["step"].step()
        return s["q_n"]
    if kind == "autograd":
        v = sv.VolumeRHS.apply(s["q"], s["geo"], s["D"], s["rho_ref"], s["theta_ref"], s["phys"])
        return v, torch.autograd.grad(v, s["q"], s["lam"])[0]
    if kind == "surface":
        return sv.surface_rhs(s["q"], s["geo"], s["nbr"], s["theta_ref"], s["phys"], out=s["out"],
                              accumulate=s["acc"])
    if kind == "rhs":
        return sv.rhs(s["q"], s["geo"], s["D"], s["nbr"], s["rho_ref"], s["theta_ref"], s["phys"],
                      out=s["out"], accumulate=s["acc"])
    if kind == "ext":
        return sv.volume_rhs_ext(s["q"], s["geo"], s["D"], s["rho_ref"], s["theta_ref"], s["phys"],
                                 dirs=s["dirs"], out=s["out"], accumulate=s["acc"])
    call = sv.volume_rhs_affine if kind == "affine" else sv.volume_rhs
    return call(s["q"], s["geo"], s["D"], s["rho_ref"], s["theta_ref"], s["phys"], out=s["out"],
                accumulate=s["acc"])


# ---------------------------------------------------------------------------
# The work of a pass
# ---------------------------------------------------------------------------
def _volume_work(case, nq, ne, nf=5, ndirs=3, geo=10, acc=False):
    """Bytes and operations of one volume term over ne elements of order nq."""
    nodes, size = ne * nq ** 3, 4 if case["f32"] else 8
    values = nf * (3 if acc else 2) + (1 if case["ref"] else 0)
    nbytes = nodes * (values * size + (8 if case["ref"] else 0))
    nbytes += (ne * 10 if geo == 0 else nodes * geo) * size
    flops = nodes * (2 * nf * ndirs * nq + ndirs * (7 + 4 * nf) + nf * 2 + 20)
    return nbytes, flops


def work(case):
    kind, size = case["kind"], 4 if case["f32"] else 8
    if kind in ("batch", "rk3"):
        both = [_volume_work(case, int(t), case["ne"]) for t in case["orders"].split()]
        nbytes, flops = sum(b for b, _ in both), sum(f for _, f in both)
        if kind == "rk3":    # three stages, two of which read q_n besides
            values = 5 * case["ne"] * sum(int(t) ** 3 for t in case["orders"].split())
            nbytes, flops = 3 * nbytes + 2 * values * size, 3 * flops + 3 * 6 * values
        return dict(bytes=nbytes, flops=flops)
    nq = case["nq"]
    ne = case["ne"] if "ne" in case else case["nx"] * case["ny"] * case["nz"]
    if kind in ("rhs", "surface"):
        face = 6 * nq * nq * ne
        if kind == "rhs":
            nbytes, flops = _volume_work(case, nq, ne, acc=case["acc"])
            return dict(bytes=nbytes + 24 * ne, flops=flops + 100 * face)
        edge = (nq ** 3 - max(0, nq - 2) ** 3) * ne
        values = edge * (6 + (10 if case["acc"] else 0)) + 3 * face
        values += 0 if case["acc"] else 5 * nq ** 3 * ne
        return dict(bytes=values * size + (8 * edge if case["ref"] else 0) + 24 * ne,
                    flops=120 * face)
    if kind == "ext":
        nbytes, flops = _volume_work(case, nq, ne, case["nf"], 3 if case["rst"] else 2,
                                     10 if case["rst"] else 7, case["acc"])
    elif kind == "affine":
        nbytes, flops = _volume_work(case, nq, ne, geo=0, acc=case["acc"])
    else:
        nbytes, flops = _volume_work(case, nq, ne, acc=case.get("acc", False))
    if kind == "autograd":
        nodes = ne * nq ** 3
        nbytes += 25 * nodes * size
        flops += nodes * (30 * nq + 150)
    return dict(bytes=nbytes, flops=flops)


# ---------------------------------------------------------------------------
# The same results in 64 bits, by plain torch
# ---------------------------------------------------------------------------
def _eos(theta, phys):
    return phys[0] * (phys[2] * theta / phys[0]) ** phys[1]


def _along(mat, f, d, nq):
    """mat applied along reference direction d of nodal fields f[..., m]."""
    if d == 0:
        g = torch.matmul(f.reshape(-1, nq), mat.t().contiguous())
    elif d == 1:
        g = torch.matmul(mat, f.reshape(-1, nq, nq))
    else:
        g = torch.matmul(mat, f.reshape(-1, nq, nq * nq))
    return g.reshape(f.shape)


def _velocity(b, d):
    geo, q = b["geo"], b["q"]
    return sum(geo[:, 3 * d + a, None] * q[:, 1 + a, None] for a in range(3)) / q[:, :1]


def _exact_volume(b, phys, ndirs=3):
    """Eq. (volterm) with the gravity source, FP64."""
    q, geo, nq = b["q"], b["geo"], b["D"].shape[0]
    p = _eos(q[:, 4], phys)
    if b["theta_ref"] is not None:
        p = p - _eos(b["theta_ref"], phys)
    out = torch.zeros_like(q)
    for d in range(ndirs):
        f = q * _velocity(b, d)
        for a in range(3):
            f[:, 1 + a] += geo[:, 3 * d + a] * p
        out += _along(b["D"], f, d, nq)
    out *= -geo[:, 9:10]
    out[:, 3] -= phys[3] * (q[:, 0] - (b["rho_ref"] if b["rho_ref"] is not None else 0.0))
    return out


def _face(nq, d, side, dev):
    m = torch.arange(nq ** 3, device=dev)
    return m[(m // nq ** d) % nq == (nq - 1 if side else 0)]


def _exact_surface(b, every, phys, lo):
    """The face term of the elements b (elements lo.. of `every`), FP64."""
    q, geo = b["q"], b["geo"]
    ne, nq = every["q"].shape[0], b["nq"]
    out = torch.zeros_like(q)
    for d in range(3):
        for side in (0, 1):
            own, other = _face(nq, d, side, q.device), _face(nq, d, 1 - side, q.device)
            to = every["nbr"][lo:lo + q.shape[0], 2 * d + side].long()
            inside = (to >= 0) & (to < ne)
            to = torch.where(inside, to, 0)
            n = (1.0 if side else -1.0) * geo[:, 3 * d:3 * d + 3][:, :, own]
            size = n.square().sum(dim=1).sqrt()
            sides = []
            for state, ref in (
                    (q[:, :, own], None if b["theta_ref"] is None else b["theta_ref"][:, own]),
                    (every["q"][:, :, other][to], None if b["theta_ref"] is None
                     else every["theta_ref"][:, other][to])):
                full = _eos(state[:, 4], phys)
                p = full if ref is None else full - _eos(ref, phys)
                un = (n * state[:, 1:4]).sum(dim=1) / state[:, 0]
                flux = state * un[:, None]
                flux[:, 1:4] += n * p[:, None]
                speed = un.abs() / size + (phys[1] * full / state[:, 0]).sqrt()
                sides.append((state, flux, speed))
            (qm, fm, sm), (qp, fp, sp) = sides
            jump = 0.5 * (fp - fm) - 0.5 * (torch.maximum(sm, sp) * size)[:, None] * (qp - qm)
            jump = jump * inside[:, None, None]
            out[:, :, own] -= geo[:, 9:10][:, :, own] * (0.5 * nq * (nq - 1)) * jump
    return out


def _exact_adjoint(b, phys):
    """(dv/dq)^T lam, FP64."""
    q, geo, nq = b["q"], b["geo"], b["D"].shape[0]
    w = -geo[:, 9:10] * b["lam"]
    dt = b["D"].t().contiguous()
    dp = phys[1] * _eos(q[:, 4], phys) / q[:, 4]
    mu = torch.zeros_like(q)
    for d in range(3):
        g = _along(dt, w, d, nq)
        vd = _velocity(b, d)
        work_d = (g[:, 1:] * q[:, 1:]).sum(dim=1)
        mu[:, 0] -= vd[:, 0] * work_d / q[:, 0]
        mu[:, 1:] += vd * g[:, 1:]
        for a in range(3):
            mu[:, 1 + a] += geo[:, 3 * d + a] * (g[:, 0] + work_d / q[:, 0])
            mu[:, 4] += dp * geo[:, 3 * d + a] * g[:, 1 + a]
    mu[:, 0] -= phys[3] * b["lam"][:, 3]
    return mu


CHUNK = 1 << 21     # nodes evaluated at a time


def _elementwise(b, nq, fn):
    """fn over chunks of the elements of b, the results joined."""
    per = max(1, CHUNK // nq ** 3)
    parts = []
    for lo in range(0, b["q"].shape[0], per):
        c = {k: (v[lo:lo + per].double() if k not in ("D", "nbr") and torch.is_tensor(v) else v)
             for k, v in b.items()}
        c["D"], c["nq"] = b["D"].double(), nq
        if c["geo"].dim() == 2:
            c["geo"] = c["geo"][:, :, None].expand(-1, -1, nq ** 3)
        parts.append(fn(c, lo))
    return torch.cat(parts)


def exact(case, seed):
    blocks, phys, kind = _inputs(case, seed), _phys(case), case["kind"]
    if kind == "batch":
        return [_elementwise(b, b["D"].shape[0], lambda c, lo: _exact_volume(c, phys))
                for b in blocks]
    if kind == "rk3":
        def step(c, lo):
            q0 = c["q"]
            for a, b in ((0.0, 1.0), (0.75, 0.25), (1.0 / 3.0, 2.0 / 3.0)):
                c["q"] = a * q0 + b * (c["q"] + RK_DT * _exact_volume(c, phys))
            return c["q"]
        return torch.cat([_elementwise(b, b["D"].shape[0], step).reshape(-1) for b in blocks])
    b, nq = blocks[0], case["nq"]
    if kind == "autograd":
        return (_elementwise(b, nq, lambda c, lo: _exact_volume(c, phys)),
                _elementwise(b, nq, lambda c, lo: _exact_adjoint(c, phys)))
    every = dict(b, q=b["q"].double())

    def one(c, lo):
        if kind == "surface":
            v = _exact_surface(c, every, phys, lo)
        else:
            v = _exact_volume(c, phys, 3 if case.get("rst", True) else 2)
            if kind == "rhs":
                v = v + _exact_surface(c, every, phys, lo)
        return v + c["out"] if case["acc"] else v
    return _elementwise(b, nq, one)
