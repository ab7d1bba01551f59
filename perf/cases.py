"""Performance cases of the long-range step: the calls that programs on top of
this library make, with the sizes of its own workloads.

A case is one of four kinds:
  step     one PPPM step (energy, forces on ions and Wannier centroids, virial)
           through Plan.compute, or through compute_noalloc ("noalloc");
  grad     one step and its backward through dplr_long_range, as a model that
           differentiates the energy calls it;
  correct  the learned correction of one frame (Mlp.forward);
  train    one training step of the correction network (Mlp.train_step).

listed() holds the standing workloads, draw() takes others from the same
ranges, prepare() builds what a program holds before the call, run() is one
call, work() its least bytes and operations, and exact() the same result in
64-bit PyTorch without the library.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2504_15508_amd as dl
from paper_2504_15508_amd import learned

BETA = 0.4            # Gaussian width, 1/Angstrom
COULOMB = 14.399645   # eV Angstrom / e^2
WATER_DENSITY = 0.0334
ALIAS = 2             # the plans' default alias range
CUTOFF, OUT_SCALE = 4.0, 0.01
LATE_LR = 1e-6        # learning rate near the end of the cosine schedule
SIZES_235 = sorted({2 ** a * 3 ** b * 5 ** c for a in range(8) for b in range(5) for c in range(4)
                    if 8 <= 2 ** a * 3 ** b * 5 ** c <= 125})


def _step(name, waters, box, mesh, order=5, precision="fp32", kind="step", diff="ik", pairs=0, noalloc=False):
    bx = (box,) * 3 if not isinstance(box, (tuple, list)) else box
    m = (mesh,) * 3 if isinstance(mesh, int) else mesh
    return {"name": name, "kind": kind, "waters": waters, "pairs": pairs,
            "lx": float(bx[0]), "ly": float(bx[1]), "lz": float(bx[2]),
            "kx": m[0], "ky": m[1], "kz": m[2], "order": order, "precision": precision, "diff": diff,
            "noalloc": noalloc}


def listed():
    return [
        # the smallest system a program differentiates through: 64 waters in
        # double precision, energy and gradient
        _step("water64_fp64_m32_grad", 64, 12.42, 32, precision="fp64", kind="grad"),
        # the precision study's largest grid: 128 waters, 12 x 18 x 12
        _step("water128_fp64_12x18x12", 128, 16.0, (12, 18, 12), precision="fp64"),
        # a training box's fine mesh (order 8), served without a plan
        _step("water1128_fp32_m32_p8_noalloc", 1128, 32.325, 32, order=8, noalloc=True),
        # a mid-sized MD box
        _step("water4096_fp32_m64", 4096, 49.7, 64),
        # the benchmark system: 216,576 atoms + 72,192 centroids
        _step("water72192_fp32_m128", 72192, 129.3, 128),
        # ... at the order that reaches 1e-4 in the forces
        _step("water72192_fp32_m128_p8", 72192, 129.3, 128, order=8),
        # ... with analytic differentiation
        _step("water72192_fp32_m128_ad", 72192, 129.3, 128, diff="ad"),
        # ... in double precision
        _step("water72192_fp64_m128", 72192, 129.3, 128, precision="fp64"),
        # ... on a mesh that is not a power of two (1.08 A spacing)
        _step("water72192_fp32_m120", 72192, 129.3, 120),
        # the largest system: 1.2 M charges of an ionic solution, forward and backward
        _step("ionic306000_fp32_m256_grad", 300000, 208.5, 256, kind="grad", pairs=3000),
        # the learned correction of one frame of the benchmark system
        {"name": "correct_water72192", "kind": "correct", "waters": 72192, "pairs": 0,
         "lx": 129.3, "ly": 129.3, "lz": 129.3},
        # one training step on a training box (residual of 16^3 order 5 against 32^3 order 8)
        {"name": "train_water1128", "kind": "train", "waters": 1128, "pairs": 0,
         "lx": 32.325, "ly": 32.325, "lz": 32.325},
    ]


def _loguniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "grad", "correct", "train"])
    hi = {"step": 100000, "grad": 100000, "correct": 100000, "train": 20000}[kind]
    waters = int(round(_loguniform(rng, 96 if kind in ("correct", "train") else 64, hi)))
    edge = (waters / WATER_DENSITY) ** (1.0 / 3.0)
    # cubic, or slightly stretched at the same volume
    sx, sy = (1.0, 1.0) if rng.random() < 0.5 else (rng.uniform(0.9, 1.1), rng.uniform(0.9, 1.1))
    box = [round(edge * sx, 3), round(edge * sy, 3), round(edge / (sx * sy), 3)]
    if kind in ("correct", "train"):
        return {"kind": kind, "waters": waters, "pairs": 0, "lx": box[0], "ly": box[1], "lz": box[2]}
    order = rng.choice([3, 4, 5, 5, 5, 6, 7, 8])
    precision = rng.choice(["fp32", "fp32", "fp32", "fp64"])
    h = _loguniform(rng, 0.8, 1.6)
    diff, noalloc = "ik", False
    if rng.random() < 0.65:  # powers of two, each axis its own
        top = 256 if precision == "fp32" else 128
        mesh = [min(top, max(16, 2 ** int(round(math.log2(b / h))))) for b in box]
        while math.prod(mesh) > 128 ** 3:
            mesh[mesh.index(max(mesh))] //= 2
        if rng.random() < 0.25:
            diff = "ad"
        noalloc = kind == "step" and rng.random() < 0.25
    else:
        top = 125 if precision == "fp32" else 90
        mesh = [min((s for s in SIZES_235 if s <= top), key=lambda s: abs(s - b / h)) for b in box]
        if all(k & (k - 1) == 0 and k >= 16 for k in mesh):
            mesh[0] = mesh[0] * 3 // 4
    pairs = rng.choice([0, 0, 0, max(1, waters // 100)])
    c = _step("", waters, box, tuple(mesh), order, precision, kind, diff, pairs, noalloc)
    del c["name"]
    return c


# --- inputs -----------------------------------------------------------------
def _rotations(rng, n):
    u1, u2, u3 = rng.random(n), rng.random(n), rng.random(n)
    a, b = np.sqrt(1 - u1), np.sqrt(u1)
    w, x = a * np.sin(2 * np.pi * u2), a * np.cos(2 * np.pi * u2)
    y, z = b * np.sin(2 * np.pi * u3), b * np.cos(2 * np.pi * u3)
    return np.stack([np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)], -1),
                     np.stack([2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)], -1),
                     np.stack([2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], -1)], -2)


def _system(case, seed):
    """Rigid waters (O +6, H +1, centroid -8 bound to O) and Na+/Cl- pairs on a
    jittered lattice; the ions behind the waters, as the systems package
    orders them.  Positions in the box, float64."""
    rng = np.random.default_rng([20260000, seed])
    nw, npair = case["waters"], case["pairs"]
    box = np.array([case["lx"], case["ly"], case["lz"]])
    ns = nw + 2 * npair
    m = int(math.ceil(round(ns ** (1 / 3), 9)))
    g = np.arange(m)
    sites = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3) + 0.5
    if m ** 3 > ns:
        sites = sites[np.sort(rng.permutation(m ** 3)[:ns])]
    sites = sites * (box / m) + rng.normal(0.0, 0.1, (ns, 3))
    perm = rng.permutation(ns) if npair else np.arange(ns)
    ions, o = sites[perm[:2 * npair]], sites[np.sort(perm[2 * npair:])]
    half = math.radians(104.5) / 2
    frame = np.array([[0.96 * math.sin(half), 0, 0.96 * math.cos(half)],
                      [-0.96 * math.sin(half), 0, 0.96 * math.cos(half)], [0, 0, 0.25]])
    off = np.matmul(_rotations(rng, nw)[:, None], frame[None, :, :, None])[..., 0]
    atoms = np.concatenate([np.stack([o, o + off[:, 0], o + off[:, 1]], 1).reshape(-1, 3), ions])
    q = np.concatenate([np.tile([6.0, 1.0, 1.0], nw), np.full(npair, 1.0), np.full(npair, -1.0)])

    def wrap(p):
        p = np.mod(p, box)
        return np.where(p >= box, 0.0, p)

    return wrap(atoms), q, wrap(o + off[:, 2]), np.full(nw, -8.0), box


def _params(seed):
    rng = np.random.default_rng([20261000, seed])
    p = {}
    for l, (a, b) in enumerate([(128, 64), (64, 64), (64, 64), (64, 32)], 1):
        p[f"W{l}"] = rng.normal(0.0, 1.0 / math.sqrt(a), (a, b)).astype(np.float32)
        p[f"b{l}"] = rng.normal(0.0, 0.02, b).astype(np.float32)
    p["mu"], p["inv_sigma"] = np.zeros(128, np.float32), np.ones(128, np.float32)
    return p


def _mesh(case):
    return case["kx"], case["ky"], case["kz"]


def _n(case):
    return 4 * case["waters"] + 2 * case["pairs"]


def prepare(case, seed):
    dev = torch.device("cuda", 0)
    dt = torch.float64 if case.get("precision") == "fp64" else torch.float32
    ri, qi, rw, qw, box = _system(case, seed)
    t = lambda a: torch.tensor(a, dtype=dt, device=dev)
    s = {"case": case, "box": tuple(float(b) for b in box), "x": (t(ri), t(qi), t(rw), t(qw))}
    if case["kind"] in ("step", "grad"):
        if not case["noalloc"]:
            s["plan"] = dl.Plan(_mesh(case), order=case["order"], beta=BETA, coulomb_k=COULOMB,
                                precision=case["precision"], capacity=_n(case), device=dev, diff=case["diff"])
            s["plan"].set_box(s["box"])
        if case["kind"] == "grad":
            s["leaf"] = (s["x"][0].clone().requires_grad_(), s["x"][2].clone().requires_grad_())
        return s
    net = learned.Mlp(_n(case), cutoff=CUTOFF, out_scale=OUT_SCALE, device=dev)
    net.set_params(_params(seed))
    net.norm_accumulate(s["box"], *s["x"])
    net.norm_finish()
    s["net"] = net
    if case["kind"] == "train":
        # coarse and fine meshes at the training boxes' spacings (about 2 and 1 A)
        forces = []
        for k, order in zip(_train_meshes(case), (5, 8)):
            plan = dl.Plan(k, order=order, beta=BETA, coulomb_k=COULOMB, capacity=_n(case), device=dev)
            plan.set_box(s["box"])
            _, fi, fw, _ = plan.compute(*s["x"])
            forces += [fi, fw]
            torch.cuda.synchronize()
            plan.close()
        s["base"], s["target"] = forces[:2], forces[2:]
    return s


def _train_meshes(case):
    edges = (case["lx"], case["ly"], case["lz"])
    coarse = tuple(min(64, max(16, 2 ** int(round(math.log2(e / 2.02))))) for e in edges)
    return coarse, tuple(2 * k for k in coarse)


def run(state):
    case = state["case"]
    ri, qi, rw, qw = state["x"]
    if case["kind"] == "step":
        if case["noalloc"]:
            return dl.plan.compute_noalloc(_mesh(case), state["box"], ri, qi, rw, qw, order=case["order"], beta=BETA,
                                           coulomb_k=COULOMB, diff=case["diff"])
        return state["plan"].compute(ri, qi, rw, qw)
    if case["kind"] == "grad":
        li, lw = state["leaf"]
        li.grad = lw.grad = None
        energy = dl.dplr_long_range(li, lw, qi, qw, state["plan"])
        energy.backward()
        return energy.detach(), li.grad, lw.grad, state["plan"].last_virial
    if case["kind"] == "correct":
        return state["net"].forward(state["box"], ri, qi, rw, qw)
    bi, bw = state["base"]
    ti, tw = state["target"]
    return state["net"].train_step(state["box"], ri, qi, rw, qw, ti, tw, LATE_LR, want_grad=True,
                                   ion_base=bi, wc_base=bw)


def work(case):
    n = _n(case)
    pairs = n * 36  # neighbours within the cutoff in water
    net = 128 * 64 + 2 * 64 * 64 + 64 * 32
    if case["kind"] == "correct":
        return {"bytes": 28 * n + 4 * net, "flops": pairs * 32 * 10 + 2 * n * (net + 128 * 4 + 32 * 3)}
    if case["kind"] == "train":
        return {"bytes": (16 + 24) * n + 4 * 8 * net, "flops": pairs * 32 * 10 + 6 * n * net}
    kx, ky, kz = _mesh(case)
    pts, p3, ts = kx * ky * kz, case["order"] ** 3, 8 if case["precision"] == "fp64" else 4
    ncomp = 1 if case["diff"] == "ad" else 3
    fft = 2.5 * pts * math.log2(pts) * (1 + ncomp)
    table = 8 * (kx // 2 + 1) * (ky // 2 + 1) * (kz // 2 + 1)
    return {"bytes": 7 * ts * n * (2 if case["kind"] == "grad" else 1) + table,
            "flops": fft + n * p3 * (2 + 6)}


# --- the same results in 64-bit PyTorch ---------------------------------------
def _bspline(d, p):
    """w[t] = M_p(d + p-1-t) and its derivative, t < p, for d in [0, 1)."""
    m = [torch.ones_like(d)]                      # M_1(d + i), i < 1
    prev = m
    for k in range(2, p + 1):
        prev = m
        m = []
        for i in range(k):
            a = (d + i) * prev[i] if i < k - 1 else 0.0
            b = (k - d - i) * prev[i - 1] if i > 0 else 0.0
            m.append((a + b) / (k - 1))
    w = [m[p - 1 - t] for t in range(p)]
    dm = [(prev[i] if i < p - 1 else 0.0) - (prev[i - 1] if i > 0 else 0.0) for i in range(p)]
    dw = [dm[p - 1 - t] + torch.zeros_like(d) for t in range(p)]
    return w, dw


def _pppm(pos, q, box, mesh, order, diff="ik"):
    """PPPM in float64: energy, forces and virial (xx, yy, zz, xy, xz, yz)."""
    dev, p = pos.device, order
    vol = box[0] * box[1] * box[2]
    start, w, dw = [], [], []
    for a in range(3):
        k = mesh[a]
        u = pos[:, a] * (k / box[a])
        u = u - k * torch.floor(u / k)
        u = torch.where(u >= k, u - k, u)
        av = u - 0.5 * p
        f = torch.floor(av)
        start.append(f.long() + 1)
        wa, da = _bspline(av - f, p)
        w.append(wa)
        dw.append(da)
    ix = [[torch.remainder(start[a] + t, mesh[a]) for t in range(p)] for a in range(3)]
    rows = [[(ix[0][i] * mesh[1] + ix[1][j]) * mesh[2] for j in range(p)] for i in range(p)]
    rho = torch.zeros(mesh[0] * mesh[1] * mesh[2], dtype=torch.float64, device=dev)
    for i in range(p):
        for j in range(p):
            qij = q * w[0][i] * w[1][j]
            for k in range(p):
                rho.index_add_(0, rows[i][j] + ix[2][k], qij * w[2][k])
    rho_k = torch.fft.rfftn(rho.view(*mesh))
    num = [torch.fft.fftfreq(k, 1.0 / k, dtype=torch.float64, device=dev) for k in mesh]
    num[2] = torch.fft.rfftfreq(mesh[2], 1.0 / mesh[2], dtype=torch.float64, device=dev)
    shape = [(-1, 1, 1), (1, -1, 1), (1, 1, -1)]
    # the Nyquist index counts as +K/2 in k (and as 0 where k appears once)
    num = [torch.where(2 * v.abs() == mesh[a], v.abs(), v) for a, v in enumerate(num)]
    kv = [(2 * math.pi / box[a]) * num[a].view(shape[a]) for a in range(3)]
    kd = [torch.where((2 * num[a].abs() == mesh[a]).view(shape[a]), torch.zeros_like(kv[a]), kv[a]) for a in range(3)]
    k2 = kv[0] ** 2 + kv[1] ** 2 + kv[2] ** 2
    u2, km = [], []
    for a in range(3):
        u2.append([torch.sinc((num[a] / mesh[a] + m)).pow(2 * p).view(shape[a]) for m in range(-ALIAS, ALIAS + 1)])
        km.append([(2 * math.pi / box[a]) * (num[a] + m * mesh[a]).view(shape[a]) for m in range(-ALIAS, ALIAS + 1)])
    top, den = torch.zeros_like(k2), torch.zeros_like(k2)
    na = 2 * ALIAS + 1
    for a in range(na):
        for b in range(na):
            for c in range(na):
                u = u2[0][a] * u2[1][b] * u2[2][c]
                kk = km[0][a] ** 2 + km[1][b] ** 2 + km[2][c] ** 2
                kk = torch.where(kk == 0, torch.ones_like(kk), kk)
                dot = kv[0] * km[0][a] + kv[1] * km[1][b] + kv[2] * km[2][c]
                top += dot * u * (4 * math.pi) * torch.exp(-kk / (4 * BETA ** 2)) / kk
                den += u
    zero = k2 == 0
    k2s = torch.where(zero, torch.ones_like(k2), k2)
    g = torch.where(zero, torch.zeros_like(k2), top / (k2s * den ** 2))
    wgt = torch.full((rho_k.shape[2],), 2.0, dtype=torch.float64, device=dev)
    wgt[0] = 1.0
    if mesh[2] % 2 == 0:
        wgt[-1] = 1.0
    e = g * (rho_k.real ** 2 + rho_k.imag ** 2) * wgt
    cc = torch.where(zero, torch.zeros_like(k2), 2 * (1 + k2 / (4 * BETA ** 2)) / k2s)
    pre = COULOMB / (2 * vol)
    vir = [pre * (e * (1 - cc * kv[a] ** 2)).sum() for a in range(3)]
    # off-diagonal terms of one Nyquist index cancel between +-k; those of two
    # belong to the sum on the mixed-radix meshes and are left out on the others
    pow2 = all(k & (k - 1) == 0 and k >= 16 for k in mesh)
    ny = [torch.zeros_like(kv[a]) if pow2 else kv[a] - kd[a] for a in range(3)]
    vir += [pre * (-e * cc * (kd[a] * kd[b] + ny[a] * ny[b])).sum() for a, b in ((0, 1), (0, 2), (1, 2))]
    force = torch.zeros_like(pos)
    if diff == "ad":
        phi = torch.fft.irfftn(g * rho_k, s=mesh, norm="forward").reshape(-1)
    for a in range(3):
        acc = torch.zeros_like(q)
        if diff == "ik":
            fld = torch.fft.irfftn(-1j * kd[a] * g * rho_k, s=mesh, norm="forward").reshape(-1)
            ws, scale = w, 1.0
        else:
            fld, scale = phi, -mesh[a] / box[a]
            ws = [dw[b] if b == a else w[b] for b in range(3)]
        for i in range(p):
            for j in range(p):
                wij = ws[0][i] * ws[1][j]
                for k in range(p):
                    acc += wij * ws[2][k] * fld[rows[i][j] + ix[2][k]]
        force[:, a] = (COULOMB / vol) * scale * q * acc
    return pre * e.sum(), force, torch.stack(vir)


def _descriptor(pos, q, box, rc=CUTOFF):
    """T[n][32][4] in float64 (cell search, one candidate per particle at a time)."""
    dev, n = pos.device, pos.shape[0]
    b = torch.tensor(box, dtype=torch.float64, device=dev)
    nc = [int(x // rc) for x in box]
    ci = torch.stack([torch.clamp((pos[:, a] / box[a] * nc[a]).long(), 0, nc[a] - 1) for a in range(3)], 1)
    cell = (ci[:, 2] * nc[1] + ci[:, 1]) * nc[0] + ci[:, 0]
    order = torch.argsort(cell)
    count = torch.bincount(cell, minlength=nc[0] * nc[1] * nc[2])
    begin = torch.cumsum(count, 0) - count
    out = torch.zeros(n, 32, 4, dtype=torch.float64, device=dev)
    me = torch.arange(n, device=dev)
    for off in range(27):
        d = (off % 3 - 1, off // 3 % 3 - 1, off // 9 - 1)
        o = [torch.remainder(ci[:, a] + d[a], nc[a]) for a in range(3)]
        other = (o[2] * nc[1] + o[1]) * nc[0] + o[0]
        b0, cnt = begin[other], count[other]
        for m in range(int(cnt.max())):
            i = me[cnt > m]
            j = order[b0[i] + m]
            dr = pos[j] - pos[i]
            dr = dr - b * torch.round(dr / b)
            r2 = (dr * dr).sum(1)
            keep = (r2 < rc * rc) & (r2 > 0) & (i != j)
            i, j, dr, r = i[keep], j[keep], dr[keep], r2[keep].sqrt()
            x = 2 * r / rc - 1
            cheb = [torch.ones_like(x), x]
            for _ in range(30):
                cheb.append(2 * x * cheb[-1] - cheb[-2])
            wt = q[j] * 0.5 * (1 + torch.cos(math.pi * r / rc))
            u = torch.cat([torch.ones_like(r)[:, None], dr / r[:, None]], 1)
            out[i] += (torch.stack(cheb, 1) * wt[:, None])[:, :, None] * u[:, None, :]
    return out


def _network(desc, q, par):
    """dF of every particle in float64; par: the named parameter tensors."""
    n = desc.shape[0]
    inv = torch.matmul(desc, desc[:, :4].transpose(1, 2).contiguous()).reshape(n, 128)
    mu = inv.mean(0)
    sd = ((inv ** 2).mean(0) - mu ** 2).clamp_min(0).sqrt()
    h = (inv - mu) / (sd + 1e-6 * (inv.abs().max() + 1.0))
    for l in (1, 2, 3):
        h = torch.nn.functional.silu(h @ par[f"W{l}"] + par[f"b{l}"])
    c = h @ par["W4"] + par["b4"]
    return OUT_SCALE * q[:, None] * (c[:, :, None] * desc[:, :, 1:]).sum(1)


def exact(case, seed):
    dev = torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")
    np_dt = np.float64 if case.get("precision") == "fp64" else np.float32
    ri, qi, rw, qw, box = _system(case, seed)
    n_ion = len(qi)
    box = [float(b) for b in box]
    # the call's inputs are positions rounded to its precision
    pos = torch.tensor(np.concatenate([ri, rw]).astype(np_dt).astype(np.float64), device=dev)
    q = torch.tensor(np.concatenate([qi, qw]), device=dev)
    if case["kind"] in ("step", "grad"):
        e, f, v = _pppm(pos, q, box, _mesh(case), case["order"], case["diff"])
        if case["kind"] == "grad":
            f = -f
        return e, f[:n_ion], f[n_ion:], v
    par = {k: torch.tensor(v.astype(np.float64), device=dev) for k, v in _params(seed).items()}
    box32 = [float(np.float32(b)) for b in box]
    desc = _descriptor(pos, q, box32)
    if case["kind"] == "correct":
        df = _network(desc, q, par)
        return df[:n_ion], df[n_ion:]
    names = [f"{k}{l}" for l in (1, 2, 3, 4) for k in ("W", "b")]
    for k in names:
        par[k].requires_grad_()
    coarse, fine = (_pppm(pos, q, box, k, p)[1] for k, p in zip(_train_meshes(case), (5, 8)))
    loss = ((_network(desc, q, par) - (fine - coarse)) ** 2).mean()
    grads = torch.autograd.grad(loss, [par[k] for k in names])
    return loss.detach(), torch.cat([x.reshape(-1) for x in grads])
