"""The work that programs have this library do, as cases of known size, with plain 64-bit references.

Each case is one call (or the two or three calls that belong together) through the public entry
points: Newton-CG solves in 2D and 3D for every law, homogenized tangents of one cell and of many
cells of uneven size, the adjoint density gradient through autograd, the allocation-free projection
and the stiffness surrogate's inference, training step and checked prediction.  Sizes are those of
the benchmark's workloads and of the paper's examples, or shortened forms of them (fewer cells, one
load increment), beside odd and ragged ones.
"""

import math

import numpy as np
import torch

from paper_2408_03804_amd import binding
from paper_2408_03804_amd.autograd import homogenized_objective
from paper_2408_03804_amd.batch import TangentBatcher
from paper_2408_03804_amd.surrogate import CNN, StiffnessSurrogate

DEV = "cuda:0"
CHANNELS = (1, 32, 64, 128, 256)
LAWS = {"le": ("small", "linear_elastic"), "j2": ("small", "j2_plastic"),
        "nh": ("finite", "neo_hookean"), "stvk": ("finite", "stvk")}


def listed():
    return [
        # the smallest cell of the tests and the paper's introductory one: a disk in a 31 x 31 cell, where
        # a solve is launches and host checks
        dict(name="solve_le_31x31", kind="solve", law="le", ny=31, nx=31, nz=0, incr=1, stored=0, cg=60),
        # the paper's elastoplastic example: prime axes, 10 load steps, tangent stored per Newton step
        dict(name="solve_j2_199x199", kind="solve", law="j2", ny=199, nx=199, nz=0, incr=10, stored=1, cg=130),
        # the paper's hyperelastic example: 299 = 13 * 23 points per axis
        dict(name="solve_stvk_299x299", kind="solve", law="stvk", ny=299, nx=299, nz=0, incr=1, stored=0, cg=140),
        # an ordinary 3D cell with axes of different length, none a power of two
        dict(name="solve_nh_45x50x54", kind="solve", law="nh", ny=50, nx=54, nz=45, incr=1, stored=0, cg=300),
        # one of the ten load increments of the 128^3 finite-strain benchmark
        dict(name="solve_nh_128", kind="solve", law="nh", ny=128, nx=128, nz=128, incr=1, stored=0, cg=380),
        # solve and 6 x 6 tangent of one 64^3 cell of stiff inclusions, contrast 100
        dict(name="tangent_le_64", kind="tangent", law="le", n=64, cg=1500),
        # training data for the surrogate: many 32^3 cells in shared launches
        dict(name="cells_32", kind="cells", sizes="32", each=96, cg=26000),
        # uncertainty quantification: cells of uneven size, one batch
        dict(name="cells_32_to_96", kind="cells", sizes="32,48,64,96", each=2, cg=2300),
        # one design step of a density optimisation: solve, objective and gradient on an odd grid
        dict(name="adjoint_nh_33", kind="adjoint", n=33, cg=800),
        # the projection alone, as a serving loop or a captured program calls it
        dict(name="project_60x63x50", kind="project", small=1, nz=60, ny=63, nx=50, batch=2),
        # the surrogate at its training batch, and the two members' checked prediction of a few cells
        dict(name="cnn_train_32_b256", kind="train", n=32, batch=256),
        dict(name="cnn_predict_32_b48", kind="predict", n=32, batch=48),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["solve2d", "solve2d", "solve3d", "cells", "adjoint", "project", "train", "predict"])
    if kind == "solve2d":
        law = rng.choice(["le", "j2", "nh", "stvk"])
        return dict(kind="solve", law=law, ny=log(16, 330), nx=log(16, 330), nz=0, incr=rng.choice([1, 2, 4]),
                    stored=rng.randint(0, 1), cg=120)
    if kind == "solve3d":
        return dict(kind="solve", law=rng.choice(["le", "j2", "nh", "stvk"]), ny=log(12, 100), nx=log(12, 100),
                    nz=log(12, 100), incr=1, stored=rng.randint(0, 1), cg=250)
    if kind == "cells":
        return dict(kind="cells", sizes=",".join(str(log(16, 60)) for _ in range(rng.randint(1, 2))),
                    each=rng.randint(2, 4), cg=1000)
    if kind == "adjoint":
        return dict(kind="adjoint", n=log(16, 40), cg=800)
    if kind == "project":
        return dict(kind="project", small=rng.randint(0, 1), nz=log(8, 64), ny=log(8, 64), nx=log(8, 64),
                    batch=rng.randint(1, 2))
    if kind == "train":
        return dict(kind="train", n=rng.choice([16, 32, 48]), batch=log(8, 200))
    return dict(kind="predict", n=rng.choice([16, 32, 48, 64]), batch=log(1, 300))


def shape_of(c):
    if "n" in c:
        return (c["n"],) * 3
    return (c["nz"], c["ny"], c["nx"]) if c["nz"] else (c["ny"], c["nx"])


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def random_cells(count, shape, length, fraction, gen):
    """`count` two-phase cells: white noise filtered to the correlation length (voxels), the top
    `fraction` of each cell's values in phase 1."""
    axes = tuple(range(1, len(shape) + 1))
    k2 = 0.0
    for a, n in enumerate(shape):
        f = torch.fft.rfftfreq(n, device=DEV) if a == len(shape) - 1 else torch.fft.fftfreq(n, device=DEV)
        k2 = k2 + (2.0 * math.pi * f.reshape([-1 if b == a else 1 for b in range(len(shape))])) ** 2
    w = torch.fft.rfftn(torch.randn((count,) + shape, generator=gen, device=DEV), dim=axes)
    g = torch.fft.irfftn(w * torch.exp(-0.25 * length ** 2 * k2), s=shape, dim=axes).reshape(count, -1)
    m = max(1, int(round(fraction * g.shape[1])))
    phase = torch.zeros(g.shape, dtype=torch.uint8, device=DEV)
    phase.scatter_(1, torch.topk(g, m, dim=1).indices, 1)
    return phase.reshape((count,) + shape)


def lame(E, nu=0.3):
    return [E * nu / ((1.0 + nu) * (1.0 - 2.0 * nu)), E / (2.0 * (1.0 + nu))]


def table_of(law, scale):
    if law == "nh":
        t = np.array([[2.0, 1.0], [40.0, 20.0]])
    elif law == "j2":
        t = np.array([lame(1.0) + [5e-3, 0.1], lame(1.0) + [1e-2, 0.2]])
    else:
        t = np.array([lame(1.0), lame(10.0)])
    t[:, :2] *= scale
    return t


def macro_of(law, d):
    if law == "nh":
        F = np.eye(d)
        F[0, 0] = 1.005
        return F.reshape(-1)
    if law == "stvk":
        F = np.eye(d)
        F[0, 1] = 0.1
        return F.reshape(-1)
    e = np.zeros(3 if d == 2 else 6)
    e[:2] = 0.01
    if law == "le":
        e[1] = 0.0
    return e


def inputs(c, seed):
    """The host and device arrays of a case, from its seed alone (shared with exact())."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    kind = c["kind"]
    if kind == "solve":
        shape = shape_of(c)
        phase = random_cells(1, shape, max(2.0, min(shape) / 16.0), 0.3, gen)[0]
        return dict(phase=phase, table=table_of(c["law"], rng.uniform(0.9, 1.1)), macro=macro_of(c["law"], len(shape)))
    if kind == "tangent":
        phase = random_cells(1, shape_of(c), 5.0, 0.2, gen)[0]
        return dict(phase=phase, table=np.array([lame(1.0), lame(100.0 * rng.uniform(0.9, 1.1))]),
                    macro=np.array([1.0, 0, 0, 0, 0, 0]))
    if kind == "cells":
        cells = []
        for n in [int(s) for s in c["sizes"].split(",")]:
            ph = random_cells(c["each"], (n,) * 3, float(rng.uniform(4.0, 8.0)), float(rng.uniform(0.2, 0.4)), gen)
            for i in range(c["each"]):
                E = float(rng.lognormal(0.0, 0.2))
                cells.append(dict(phase=ph[i], table=np.array([lame(E), lame(10.0 * E)])))
        return dict(cells=cells)
    if kind == "adjoint":
        shape = shape_of(c)
        rho = 0.2 + 0.8 * torch.rand(shape, generator=gen, device=DEV, dtype=torch.float64)
        return dict(phase=random_cells(1, shape, 4.0, 0.3, gen)[0], rho=rho, table=np.array([[2.0, 1.0], [10.0, 5.0]]),
                    macro=np.array([1.02, 0.01, 0, 0, 1, 0, 0, 0, 1.0]), ws=np.array([1.0, 0.5, 0, 0, 0, 0, 0, 0, 0]),
                    we=0.3, p=3.0)
    if kind == "project":
        ncomp = 6 if c["small"] else 9
        return dict(x=torch.randn((c["batch"], ncomp) + shape_of(c), generator=gen, device=DEV, dtype=torch.float64))
    phase = random_cells(c["batch"], shape_of(c), 8.0 * c["n"] / 32.0, 0.3, gen)
    E = rng.lognormal(0.0, 0.5, size=(c["batch"], 2))
    tables = np.array([[lame(a), lame(b)] for a, b in E])
    feat = np.log(E[:, 1] / E[:, 0])[:, None].astype(np.float32)
    out = dict(phase=phase, tables=tables, feat=torch.as_tensor(feat, device=DEV),
               theta=[random_params(np.random.default_rng([seed, i])) for i in range(2)])
    if kind == "train":
        out["target"] = torch.randn((c["batch"], 21), generator=gen, device=DEV)
    return out


def layers():
    """(rows, inputs) of the surrogate's six weight blocks."""
    return [(CHANNELS[i], 27 * CHANNELS[i - 1]) for i in range(1, 5)] + [(256, 257), (21, 256)]


def random_params(rng):
    out = []
    for rows, k in layers():
        lim = math.sqrt(6.0 / k)
        out += [rng.uniform(-lim, lim, size=rows * k), rng.uniform(-0.05, 0.05, size=rows)]
    return torch.as_tensor(np.concatenate(out).astype(np.float32), device=DEV)


# ---------------------------------------------------------------------------
# what a program keeps, and one pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    s = dict(case=case, **inputs(case, seed))
    kind = case["kind"]
    if kind in ("solve", "tangent"):
        kin, mat = LAWS[case["law"]]
        paper = case["law"] == "stvk"
        h = binding.FFTHomog(shape_of(case), kin, mat, 2, device=DEV, tol_newton=1e-5 if paper else 1e-10,
                             tol_cg=1e-8 if paper else 1e-10, max_newton=50, max_cg=20000,
                             k_mode=case.get("stored", 0), tangent=kind == "tangent")
        h.set_material(s["phase"], s["table"])
        h.tune_placement(reps=10)  # does nothing on grids too small for it
        s["h"] = h
    elif kind == "cells":
        s["b"] = TangentBatcher(tol_cg=1e-10, max_cg=20000, device=DEV)
        s["b"].tangents(s["cells"])  # makes and tunes the handles that the program keeps
    elif kind == "adjoint":
        s["h"] = binding.FFTHomog(shape_of(case), "finite", "neo_hookean", 2, device=DEV, tol_newton=1e-10,
                                  tol_cg=1e-11, max_newton=30, max_cg=20000, density=True)
    elif kind == "project":
        law = "le" if case["small"] else "nh"
        s["desc"] = binding.make_desc(shape_of(case), *LAWS[law], 1)
        s["out"] = torch.empty_like(s["x"])
    elif kind == "train":
        s["net"] = CNN(n=case["n"], max_batch=case["batch"], device=DEV)
        s["net"].set_params(s["theta"][0])
    else:
        sur = StiffnessSurrogate(n=case["n"], max_batch=case["batch"], device=DEV, members=2)
        for net, th in zip(sur.nets, s["theta"]):
            net.set_params(th)
        sur.fold()
        s["sur"] = sur
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "solve":
        s["h"].reset()
        out, psi, _ = s["h"].solve(s["macro"], c["incr"])
        return dict(stress=out, energy=psi, strain=s["h"].get_field(binding.FIELD_STRAIN))
    if kind == "tangent":
        s["h"].reset()
        out, psi, _ = s["h"].solve(s["macro"])
        C, _ = s["h"].tangent()
        return dict(stress=out, energy=psi, tangent=C, strain=s["h"].get_field(binding.FIELD_STRAIN))
    if kind == "cells":
        C, _ = s["b"].tangents(s["cells"])
        return np.stack(list(C))
    if kind == "adjoint":
        rho = s["rho"].clone().requires_grad_(True)
        J = homogenized_objective(rho, s["h"], s["phase"], s["table"], s["p"], s["macro"], 1, s["ws"], s["we"])
        J.backward()
        return dict(J=J.detach(), grad=rho.grad)
    if kind == "project":
        return binding.fft_homog_project_noalloc(s["desc"], s["x"], s["out"])
    if kind == "train":
        loss, grad = s["net"].loss_grad(s["phase"], s["feat"], s["target"])
        s["net"].adam_step(1e-3)
        return dict(loss=loss, grad=grad, params=s["net"].get_params())
    C, ok = s["sur"].predict_checked(s["phase"], s["tables"])
    return dict(C=C, ok=ok)


def work(c):
    """One pass at its least.  A CG iteration reads the phase (and a finite-strain or plastic state)
    and reads and writes its three vectors, `d` numbers per voxel each (the displacement that a
    compatible strain comes from); it transforms every strain component forward and back.  `cg` is
    the usual number of iterations, over all right-hand sides of a pass."""
    kind = c["kind"]
    if kind in ("train", "predict"):
        n, e, f = c["batch"], c["n"], 0
        par = sum(r * k + r for r, k in layers())
        for i in range(4):
            e //= 2
            f += 2 * e ** 3 * layers()[i][0] * layers()[i][1]
        f += sum(2 * r * k for r, k in layers()[4:])
        if kind == "train":
            return dict(bytes=n * (c["n"] ** 3 + 4 * 22) + 4 * par * 7, flops=3 * f * n)
        return dict(bytes=n * (c["n"] ** 3 + 4 * 28) + 2 * 4 * par, flops=2 * f * n)
    shapes = [(int(n),) * 3 for n in c["sizes"].split(",")] if kind == "cells" else [shape_of(c)]
    N = sum(int(np.prod(s)) for s in shapes) / len(shapes)
    d = len(shapes[0])
    small = c["small"] if kind == "project" else LAWS[c.get("law", "le" if kind == "cells" else "nh")][0] == "small"
    ncomp = (3 if d == 2 else 6) if small else d * d
    fft = 2 * ncomp * 2.5 * N * math.log2(N)
    if kind == "project":
        return dict(bytes=c["batch"] * 16 * ncomp * N, flops=c["batch"] * fft)
    state = 0 if small and c.get("law") != "j2" else 8 * ncomp
    return dict(bytes=c["cg"] * N * (1 + state + 6 * 8 * d), flops=c["cg"] * (fft + 40 * ncomp * N))


# ---------------------------------------------------------------------------
# the same results in 64 bits by plain torch
# ---------------------------------------------------------------------------
def gradient_projection(shape, small):
    """A -> compatible part of A, (..., d, d, *shape); a Nyquist index has a zero wavevector entry."""
    d = len(shape)
    xi = []
    for a in range(d):  # component a belongs to the a-th axis from the right (x fastest)
        n = shape[d - 1 - a]
        k = (torch.fft.rfftfreq(n, dtype=torch.float64, device=DEV) if a == 0
             else torch.fft.fftfreq(n, dtype=torch.float64, device=DEV)) * n
        if n % 2 == 0:
            k[n // 2] = 0.0
        xi.append((2.0 * math.pi * k).reshape([-1 if b == d - 1 - a else 1 for b in range(d)]))
    n2 = sum(x * x for x in xi)
    inv = torch.where(n2 > 0, 1.0 / torch.where(n2 > 0, n2, 1.0).sqrt(), 0.0)
    nv = [x * inv for x in xi]
    dims = tuple(range(-d, 0))

    def apply(A):
        h = torch.fft.rfftn(A, dim=dims)
        get = [[h.select(-d - 2, i).select(-d - 1, j) for j in range(d)] for i in range(d)]
        an = [sum(get[i][j] * nv[j] for j in range(d)) for i in range(d)]
        nan = sum(nv[i] * an[i] for i in range(d))
        o = [[an[i] * nv[j] + nv[i] * an[j] - nan * nv[i] * nv[j] if small else an[i] * nv[j] for j in range(d)]
             for i in range(d)]
        o = torch.stack([torch.stack(r, dim=-d - 1) for r in o], dim=-d - 2)
        return torch.fft.irfftn(o, s=shape, dim=dims)

    return apply


def stress_and_energy(law, lam, mu, F, hist=None, sy=None, H=None):
    """P and psi at F (d, d, *shape) (small strain: eps); J2: also the updated history."""
    d = F.shape[0]
    eye = torch.eye(d, dtype=F.dtype, device=F.device).reshape((d, d) + (1,) * (F.dim() - 2))
    if law == "le":
        tr = sum(F[i, i] for i in range(d))
        P = lam * tr * eye + 2.0 * mu * F
        return P, 0.5 * (P * F).sum((0, 1)), None
    if law == "stvk":
        E = 0.5 * (sum(F[k][:, None] * F[k][None] for k in range(d)) - eye)
        S = lam * sum(E[i, i] for i in range(d)) * eye + 2.0 * mu * E
        P = sum(F[:, k][:, None] * S[k][None] for k in range(d))
        return P, 0.5 * (S * E).sum((0, 1)), None
    if law == "nh":
        if d == 3:
            cof = torch.stack([torch.stack([F[(i + 1) % 3, (j + 1) % 3] * F[(i + 2) % 3, (j + 2) % 3]
                                            - F[(i + 1) % 3, (j + 2) % 3] * F[(i + 2) % 3, (j + 1) % 3]
                                            for j in range(3)]) for i in range(3)])
        else:
            cof = torch.stack([torch.stack([F[1, 1], -F[1, 0]]), torch.stack([-F[0, 1], F[0, 0]])])
        J = (F[0] * cof[0]).sum(0)
        lnJ = J.log()
        P = mu * F + (lam * lnJ - mu) * cof / J
        return P, 0.5 * mu * ((F * F).sum((0, 1)) - d) - mu * lnJ + 0.5 * lam * lnJ * lnJ, None
    ep, p = hist  # J2: the 3D return mapping on the strain with zero out-of-plane entries
    e3 = torch.zeros((3, 3) + F.shape[2:], dtype=F.dtype, device=F.device)
    pad = torch.nn.functional.pad(F.movedim((0, 1), (-2, -1)), (0, 3 - d, 0, 3 - d)).movedim((-2, -1), (0, 1))
    eye3 = torch.eye(3, dtype=F.dtype, device=F.device).reshape((3, 3) + (1,) * (F.dim() - 2))
    ee = e3 + pad - ep
    tr = sum(ee[i, i] for i in range(3))
    s = 2.0 * mu * (ee - tr / 3.0 * eye3)
    ss = (s * s).sum((0, 1))
    safe = torch.where(ss > 0, ss, 1.0)
    seq = torch.where(ss > 0, (1.5 * safe).sqrt(), 0.0)
    phi = seq - (sy + H * p)
    dp = torch.where(phi > 0, phi / (3.0 * mu + H), 0.0)
    n = 1.5 * s / torch.where(seq > 0, seq, 1.0)
    ee = ee - dp * n
    tr = sum(ee[i, i] for i in range(3))
    sig = lam * tr * eye3 + 2.0 * mu * ee
    return sig[:d, :d], 0.5 * (sig * ee).sum((0, 1)), (ep + dp * n, p + dp)


def cg(op, b, tol, batch_dims, most=20000):
    """Conjugate gradients from zero on every right-hand side of b's leading batch_dims axes."""
    dims = tuple(range(batch_dims, b.dim()))

    def dot(u, v):
        return (u * v).sum(dims, keepdim=True)

    x, r, p = torch.zeros_like(b), b.clone(), b.clone()
    rr = dot(r, r)
    stop = tol * tol * rr
    for _ in range(most):
        if not bool((rr > stop).any()):
            break
        q = op(p)
        run_ = rr > stop
        a = torch.where(run_, rr / torch.where(run_, dot(p, q), 1.0), 0.0)
        x = x + a * p
        r = r - a * q
        new = dot(r, r)
        p = r + torch.where(run_, new / torch.where(run_, rr, 1.0), 0.0) * p
        rr = torch.where(run_, new, rr)
    return x


def full_macro(macro, d, small):
    if not small:
        return np.asarray(macro, dtype=np.float64).reshape(d, d)
    e = np.zeros((d, d))
    pairs = [(0, 0), (1, 1), (0, 1)] if d == 2 else [(0, 0), (1, 1), (2, 2), (1, 2), (0, 2), (0, 1)]
    for k, (i, j) in enumerate(pairs):
        e[i, j] = e[j, i] = macro[k] if i == j else 0.5 * macro[k]
    return e


def out_vector(P, small):
    """Macro stress of voxel averages (d, d) in the entry points' order."""
    d = P.shape[0]
    if not small:
        return P.reshape(-1)
    pairs = [(0, 0), (1, 1), (0, 1)] if d == 2 else [(0, 0), (1, 1), (2, 2), (1, 2), (0, 2), (0, 1)]
    return np.array([P[i, j] for i, j in pairs])


def newton(law, shape, phase, table, macro, incr, rho=None, simp=0.0, tol=1e-12):
    """Converged F, the law at it (F -> P, psi, history), K : dF at it, the projection."""
    small = LAWS[law][0] == "small"
    d = len(shape)
    dims = tuple(range(2, 2 + d))
    t = torch.as_tensor(table, dtype=torch.float64, device=DEV)
    lam, mu = t[:, 0][phase.long()], t[:, 1][phase.long()]
    if rho is not None:
        lam, mu = lam * rho ** simp, mu * rho ** simp
    extra, hist = {}, None
    if law == "j2":
        extra = dict(sy=t[:, 2][phase.long()], H=t[:, 3][phase.long()])
        hist = (torch.zeros((3, 3) + shape, dtype=torch.float64, device=DEV),
                torch.zeros(shape, dtype=torch.float64, device=DEV))
    G = gradient_projection(shape, small)
    target = full_macro(macro, d, small)
    start = np.zeros((d, d)) if small else np.eye(d)
    F = torch.as_tensor(start, device=DEV).reshape((d, d) + (1,) * d).expand((d, d) + shape).clone()
    for n in range(incr):
        F = F + torch.as_tensor((target - start) / incr, device=DEV).reshape((d, d) + (1,) * d)

        def law_at(f):
            return stress_and_energy(law, lam, mu, f, hist, **extra)

        for _ in range(40):
            b = -G(law_at(F)[0])
            if float(b.norm()) <= 1e-14 * float(law_at(F)[0].norm()):
                break
            at = F
            x = cg(lambda v: G(torch.func.jvp(lambda f: law_at(f)[0], (at,), (v,))[1]), b, tol, 0)
            F = F + x
            if float(x.norm()) <= 1e-12 * float(F.norm()):
                break
        if law == "j2" and n + 1 < incr:
            hist = law_at(F)[2]
    end = F

    def K(v):
        return torch.func.jvp(lambda f: law_at(f)[0], (end,), (v,))[1]

    return F, law_at, K, G, dims


def tangent_of(phase, table):
    """6 x 6 tangent of a linear elastic cell."""
    shape = tuple(phase.shape)
    t = torch.as_tensor(table, dtype=torch.float64, device=DEV)
    lam, mu = t[:, 0][phase.long()], t[:, 1][phase.long()]
    G = gradient_projection(shape, True)
    eye = torch.eye(3, dtype=torch.float64, device=DEV).reshape(1, 3, 3, 1, 1, 1)
    E = torch.stack([torch.as_tensor(full_macro(row, 3, True), device=DEV) for row in np.eye(6)])
    E = E.reshape((6, 3, 3, 1, 1, 1))

    def K(v):
        return lam * sum(v[:, i, i] for i in range(3))[:, None, None] * eye + 2.0 * mu * v

    full = E + cg(lambda v: G(K(v)), -G(K(E + torch.zeros((1, 1, 1) + shape, dtype=torch.float64, device=DEV))), 1e-12, 1)
    s = K(full)
    return np.array([[float((full[i] * s[j]).sum()) / phase.numel() for j in range(6)] for i in range(6)])


def conv_forward(theta, phase, feat):
    """(B, 21) of the network for flat 64-bit parameters."""
    def gelu(x):
        return 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))

    at, a = 0, phase.double()[..., None]
    for l, (rows, k) in enumerate(layers()):
        W, b = theta[at:at + rows * k].reshape(rows, k), theta[at + rows * k:at + rows * k + rows]
        at += rows * k + rows
        if l < 4:
            ci = k // 27
            p = torch.cat([a[:, -1:], a], 1)
            p = torch.cat([p[:, :, -1:], p], 2)
            p = torch.cat([p[:, :, :, -1:], p], 3)
            m = a.shape[1] // 2
            pre = b
            for tap in range(27):
                z, y, x = tap // 9, tap // 3 % 3, tap % 3
                v = p[:, z:z + 2 * m:2, y:y + 2 * m:2, x:x + 2 * m:2]
                pre = pre + (v.reshape(-1, ci) @ W[:, tap * ci:(tap + 1) * ci].T).reshape(v.shape[:-1] + (rows,))
            a = gelu(pre)
        elif l == 4:
            a = gelu(torch.cat([a.mean((1, 2, 3)), feat.double()], 1) @ W.T + b)
        else:
            return a @ W.T + b


def reference_bounds(tables, f):
    """Reuss stiffness (upper triangle) and the size of the gap to the Voigt one, per cell."""
    up = [(i, j) for i in range(6) for j in range(i, 6)]

    def iso(l, m):
        C = np.zeros((6, 6))
        C[:3, :3] = l
        C[range(6), range(6)] += np.array([2 * m] * 3 + [m] * 3)
        return C

    ref, gap = [], []
    for (a, b), v in zip(tables, f):
        V = iso((1 - v) * a[0] + v * b[0], (1 - v) * a[1] + v * b[1])
        k = 1.0 / ((1 - v) / (a[0] + 2 * a[1] / 3) + v / (b[0] + 2 * b[1] / 3))
        m = 1.0 / ((1 - v) / a[1] + v / b[1])
        R = iso(k - 2 * m / 3, m)
        ref.append([R[i, j] for i, j in up])
        gap.append(np.linalg.norm(V - R))
    return np.array(ref), np.array(gap)


def exact(case, seed):
    s = inputs(case, seed)
    kind = case["kind"]
    if kind in ("solve", "tangent"):
        shape = shape_of(case)
        small = LAWS[case["law"]][0] == "small"
        if case["law"] == "stvk" and kind == "solve":
            tol = 1e-10
        else:
            tol = 1e-12
        F, law, _, _, dims = newton(case["law"], shape, s["phase"], s["table"], s["macro"], case.get("incr", 1), tol=tol)
        P, psi, _ = law(F)
        res = dict(stress=out_vector(P.mean(dims).cpu().numpy(), small), energy=float(psi.mean()), strain=F)
        if kind == "tangent":
            res["tangent"] = tangent_of(s["phase"], s["table"])
        return res
    if kind == "cells":
        return np.stack([tangent_of(c["phase"], c["table"]) for c in s["cells"]])
    if kind == "adjoint":
        F, law, K, G, dims = newton("nh", shape_of(case), s["phase"], s["table"], s["macro"], 1, s["rho"], s["p"])
        P, psi, _ = law(F)
        W = torch.as_tensor(s["ws"].reshape(3, 3), device=DEV).reshape(3, 3, 1, 1, 1)
        g = s["we"] * P + K(W.expand(F.shape))
        x = cg(lambda v: G(K(v)), -G(g), 1e-12, 0)
        grad = s["p"] / (s["phase"].numel() * s["rho"]) * (s["we"] * psi + ((W + x) * P).sum((0, 1)))
        return dict(J=(s["we"] * psi.mean() + (W * P).sum((0, 1)).mean()), grad=grad)
    if kind == "project":
        d, x = 3, s["x"]
        G = gradient_projection(shape_of(case), bool(case["small"]))
        if not case["small"]:
            return G(x.reshape((case["batch"], d, d) + shape_of(case))).reshape(x.shape)
        r = math.sqrt(0.5)
        rows = [[x[:, 0], r * x[:, 5], r * x[:, 4]], [r * x[:, 5], x[:, 1], r * x[:, 3]],
                [r * x[:, 4], r * x[:, 3], x[:, 2]]]
        y = G(torch.stack([torch.stack(q, 1) for q in rows], 1))
        return torch.stack([y[:, 0, 0], y[:, 1, 1], y[:, 2, 2], y[:, 1, 2] / r, y[:, 0, 2] / r, y[:, 0, 1] / r], 1)
    if kind == "train":
        th = s["theta"][0].double().requires_grad_(True)
        loss = ((conv_forward(th, s["phase"], s["feat"]) - s["target"].double()) ** 2).mean()
        loss.backward()
        g = th.grad
        return dict(loss=float(loss.detach()), grad=g, params=th.detach() - 1e-3 * g / (g.abs() + 1e-8))
    f = s["phase"].reshape(case["batch"], -1).double().mean(1).cpu().numpy()
    ref, gap = reference_bounds(s["tables"], f)
    with torch.no_grad():
        y = 0.5 * sum(conv_forward(t.double(), s["phase"], s["feat"]) for t in s["theta"])
    return dict(C=torch.as_tensor(ref, device=DEV) + torch.as_tensor(gap, device=DEV)[:, None] * y, ok=None)
