"""Performance cases of the transport sweep: what its users run, over the range they run it at.

A case names one call sequence (`do`) on one synthetic input:

    forward   a sweep on graphs that are kept (many sweeps per mesh: source iteration loops,
              parameter studies, radiation steps between mesh updates)
    grad      the same through SweepFunction, forward and backward
    build     graphs for a new mesh, then one sweep (a moving mesh changes at every step)
    step      graphs for a new mesh, a sweep that keeps what the adjoint needs, and the adjoint
              (the step that bench.py times)
    ionise    photoionisation time steps: exponential-law sweep and chemistry

Meshes are Voronoi tiles (periodic, made by synth/) repeated tx x ty x tz times, so that large
grids are quick to make; a vacuum box cuts the faces that leave it.  Points are uniform, a
jittered lattice or clustered (lognormal density); "lattice" is a plain cubic grid.
"""
import math

import numpy as np
import torch

import paper_2207_12848_amd as sw
from synth import mesh as synth_mesh
from synth import workloads
from synth.directions import direction_set

KPC_CM = 3.0856775814913673e21
HII = dict(n_H=1e-3, sigma_H=5.38e-18, alpha_B=2.59e-13, photon_rate=1e49,
           length_unit=12.8 * KPC_CM, courant=1.0)
GROUP_SCALE = (1.0, 0.3, 0.1, 0.03, 0.01, 0.003)

DEFAULT = dict(do="forward", mesh="uniform", n=4096, tx=1, ty=1, tz=1, meshes=1, n_hi=0, periodic=False,
               D=84, G=1, law="upwind", scheme="area", albedo=0.0, n_scat=1, n_pbc=1, merge=False,
               validate=False, sources=100, steps=1)


def _case(**kw):
    return dict(DEFAULT, **kw)


def listed():
    return [
        # a first look or a unit test: a few thousand cells and the octant directions; launches
        # and the chain of levels are all there is
        _case(name="sweep_4k_8dirs", D=8, sources=1),
        # the whole path at that size as a first call makes it: mesh check on (the default),
        # graphs, sweep, adjoint
        _case(name="step_4k_8dirs_checked", do="step", D=8, sources=1, validate=True),
        # the R-type test's 32^3 run: four time steps from a half-grown ionised sphere
        _case(name="ionise_32", do="ionise", mesh="lattice", n=32, law="exp", steps=4, sources=1),
        # its resolution study at 128^3 cells, regular levels thousands of tasks wide
        _case(name="ionise_128", do="ionise", mesh="lattice", n=128, law="exp", steps=2, sources=1),
        # the scaling workload: 64^3 jittered cells, the paper's 84 directions, one bin
        _case(name="sweep_64_84dirs", mesh="jitter", n=32768, tx=2, ty=2, tz=2),
        # the same grid when the mesh has moved: graphs anew, then the sweep
        _case(name="build_64_84dirs", do="build", mesh="jitter", n=32768, tx=2, ty=2, tz=2),
        # an ordinary mesh handed over with the default checks on
        _case(name="build_50k_checked", do="build", n=16807, tx=3, D=48, validate=True),
        # fitting opacities: gradients at 64^3 cells, 48 directions
        _case(name="grad_64_48dirs", do="grad", mesh="jitter", n=32768, tx=2, ty=2, tz=2, D=48, sources=50),
        # scattering: uneven independent meshes, 24 directions, source iteration
        _case(name="scatter_uneven", meshes=12, n=512, n_hi=8192, tx=2, ty=2, tz=2, D=24, albedo=0.5,
              n_scat=10, sources=16),
        # direction-conserving transport with the exponential law, three bins, ragged sizes
        _case(name="aligned_exp_3groups", n=6151, tx=3, ty=2, D=47, G=3, law="exp", scheme="aligned"),
        # periodic box with scattering, merged iterations, two bins, with gradients
        _case(name="periodic_merged_grad", do="grad", mesh="cluster", n=15013, tx=2, periodic=True, D=24,
              G=2, albedo=0.25, n_scat=4, n_pbc=3, merge=True),
        # the benchmark's step: a clustered periodic box of 2M cells, 84 directions, four bins,
        # three periodic passes, forward and adjoint on new graphs
        _case(name="step_2m_84dirs_4groups", do="step", mesh="cluster", n=32768, tx=4, ty=4, tz=4,
              periodic=True, G=4, n_pbc=3, sources=10000),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    do = rng.choice(["forward", "forward", "grad", "build", "step", "ionise"])
    if do == "ionise":
        return _case(do=do, mesh="lattice", n=logint(20, 112), D=rng.choice([24, 48, 84]), law="exp",
                     steps=rng.randint(1, 4), sources=1)
    c = _case(do=do, mesh=rng.choice(["uniform", "jitter", "cluster"]), n=logint(2500, 24000),
              tx=rng.randint(1, 4), ty=rng.randint(1, 3), tz=rng.randint(1, 2), periodic=rng.random() < 0.4,
              D=rng.choice([8, logint(11, 96), logint(24, 96), 84]), G=rng.choice([1, 1, 2, 3, 4, 5]),
              law=rng.choice(["upwind", "upwind", "exp"]), scheme=rng.choice(["area", "area", "area", "aligned"]),
              validate=do in ("build", "step") and rng.random() < 0.4, sources=logint(1, 1000))
    if do == "forward" and rng.random() < 0.3:
        c.update(mesh="uniform", meshes=rng.randint(2, 10), n=logint(300, 1200), n_hi=logint(2000, 8000))
    if c["periodic"]:
        c["n_pbc"] = rng.randint(1, 4)
    if do in ("forward", "grad") and rng.random() < 0.4:
        c.update(albedo=rng.choice([0.25, 0.5, 0.75]), n_scat=rng.randint(2, 5), merge=rng.random() < 0.5)
        c["D"] = min(c["D"], 48)
    return c


# ------------------------------------------------------------------------------- inputs
def _tile(case, n, rng):
    """Periodic Voronoi tile of about n cells and each cell's relative opacity."""
    if case["mesh"] == "jitter":
        s = max(4, round(n ** (1 / 3)))
        m = workloads.jittered_lattice_mesh(s, rng, periodic=True)
        dens = None
    elif case["mesh"] == "cluster":
        rho = workloads.lognormal_density_grid(8, 2.0, rng)
        m = synth_mesh.voronoi_mesh(workloads.clustered_points(n, rho, rng), periodic=True)
        dens = workloads.density_at(m["points"], rho)
    else:
        m = workloads.uniform_mesh(n, rng, periodic=True)
        dens = None
    return m, dens


def _repeat(m, reps, periodic):
    """The mesh of reps[0] x reps[1] x reps[2] copies of a periodic tile, as device tensors;
    the longest side of the box is 1."""
    dev = "cuda"
    n, nf = len(m["cell_volume"]), len(m["face_nbr"])
    h = 1.0 / max(reps)
    code = torch.as_tensor(m["face_shift"], device=dev).long() + 13
    sh = torch.stack([code // 9 - 1, code // 3 % 3 - 1, code % 3 - 1])  # [3, nf] image of the neighbour
    nbr = torch.as_tensor(m["face_nbr"], device=dev).long()
    twin = torch.as_tensor(m["face_twin"], device=dev).long()
    area = torch.as_tensor(m["face_area"], device=dev) * h * h
    normal = torch.as_tensor(m["face_normal"], device=dev).reshape(-1)
    ptr = torch.as_tensor(m["face_ptr"], device=dev)
    T = reps[0] * reps[1] * reps[2]
    t = torch.arange(T, device=dev)
    at = torch.stack([t // (reps[1] * reps[2]), t // reps[2] % reps[1], t % reps[2]])  # [3, T]
    nb, tw, out = [], [], []
    for k in range(T):
        to = at[:, k:k + 1] + sh
        size = torch.tensor(reps, device=dev)[:, None]
        o = torch.div(to, size, rounding_mode="floor").clamp(-1, 1)
        w = to % size
        wid = (w[0] * reps[1] + w[1]) * reps[2] + w[2]
        wrapped = (o != 0).any(0)
        nbk, twk = wid * n + nbr, wid * nf + twin
        ck = (o[0] + 1) * 9 + (o[1] + 1) * 3 + o[2] + 1 - 13
        if not periodic:
            nbk, twk = torch.where(wrapped, -1, nbk), torch.where(wrapped, -1, twk)
        nb.append(nbk.int())
        tw.append(twk.int())
        out.append(ck.to(torch.int8))
    fp = (ptr[:-1][None, :] + t[:, None] * nf).reshape(-1)
    return dict(face_ptr=torch.cat([fp, torch.tensor([T * nf], device=dev)]).contiguous(),
                face_nbr=torch.cat(nb), face_twin=torch.cat(tw), face_shift=torch.cat(out) if periodic else None,
                face_area=area.repeat(T), face_normal=normal.repeat(T),
                cell_volume=(torch.as_tensor(m["cell_volume"], device=dev) * h ** 3).repeat(T))


def _inputs(case, seed):
    """Meshes (device tensors), directions, kappa and emission [C, G] (device, FP32)."""
    rng = np.random.default_rng([2207, 12848, int(seed) % (1 << 31)])
    G = case["G"]
    if case["mesh"] == "lattice":
        m = synth_mesh.lattice_mesh(case["n"])
        C = case["n"] ** 3
        em = np.zeros((C, 1), np.float32)
        em[case["n"] // 2 * (1 + case["n"] * (1 + case["n"]))] = 1.0
        m = {k: torch.as_tensor(m[k], device="cuda") for k in ("face_ptr", "face_nbr", "face_twin", "face_area",
                                                                "face_normal", "cell_volume")}
        return [dict(m, face_shift=None)], direction_set(case["D"]), None, torch.as_tensor(em, device="cuda")
    meshes, kap, em = [], [], []
    M = case["meshes"]
    for i in range(M):
        n = case["n"] if M == 1 else round(case["n"] * (case["n_hi"] / case["n"]) ** (i / (M - 1)))
        tile, dens = _tile(case, n, rng)
        mesh = _repeat(tile, (case["tx"], case["ty"], case["tz"]), case["periodic"])
        V = mesh["cell_volume"].cpu().numpy()
        C = len(V)
        if dens is None:
            k = workloads.lognormal_kappa(V, rng, 1.0, 10.0)
        else:
            k = workloads.scale_to_mean_tau(np.tile(dens, C // len(dens)), V, 10.0)
        cells, lum = workloads.point_sources(C, case["sources"], rng)
        e = np.zeros((C, G), np.float32)
        e[cells] = lum[:, None]
        meshes.append(mesh)
        kap.append((k[:, None] * np.array(GROUP_SCALE[:G])).astype(np.float32))
        em.append(e)
    return (meshes, direction_set(case["D"]), torch.as_tensor(np.concatenate(kap), device="cuda"),
            torch.as_tensor(np.concatenate(em), device="cuda"))


def _opts(case):
    o = dict(boundary="periodic" if case["periodic"] else "vacuum", law=case["law"])
    if case["periodic"]:
        o.update(n_pbc=case["n_pbc"])
    if case["n_scat"] > 1:
        o.update(albedo=case["albedo"], n_scat=case["n_scat"])
        if case["periodic"]:
            o.update(merge=case["merge"])
    return o


def _hii(case, seed):
    """Parameters and a partly ionised state: a sphere of the seed's radius with a smooth edge."""
    rng = np.random.default_rng([51, int(seed) % (1 << 31)])
    n = case["n"]
    p = dict(HII, dt_max=0.05 / (HII["alpha_B"] * HII["n_H"]))
    x = (torch.arange(n, device="cuda", dtype=torch.float64) - n // 2) / n
    r = (x[:, None, None] ** 2 + x[None, :, None] ** 2 + x[None, None, :] ** 2).sqrt().reshape(-1)
    edge = torch.special.expit((r - rng.uniform(0.12, 0.3)) * n * rng.uniform(1.0, 2.0))
    return p, 2e-4 + (1 - 2e-4) * edge


def _loss_grads(case, seed, C):
    g = torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 31))
    return (torch.rand((C, case["G"]), generator=g, device="cuda"),
            torch.rand((C, case["G"]), generator=g, device="cuda") / (4 * math.pi))


def prepare(case, seed):
    meshes, dirs, kappa, emission = _inputs(case, seed)
    s = dict(case=case, dirs=dirs, kappa=kappa, emission=emission, opts=_opts(case))
    if case["do"] in ("forward", "grad", "ionise"):
        s["dag"] = sw.build_dag(meshes, dirs, validate=case["validate"], scheme=case["scheme"])
    else:
        s["meshes"] = meshes
    if case["do"] == "ionise":
        s["params"], s["neutral"] = _hii(case, seed)
    if case["do"] in ("grad", "step"):
        s["gJ"], s["gA"] = _loss_grads(case, seed, kappa.shape[0])
    if case["do"] == "grad":
        kappa.requires_grad_(True)
        emission.requires_grad_(True)
    return s


def run(s):
    case, o = s["case"], s["opts"]
    do = case["do"]
    if do == "forward":
        return sw.forward(s["dag"], s["kappa"], s["emission"], **o)
    if do == "grad":
        J, A, tot = sw.SweepFunction.apply(s["kappa"], s["emission"], s["dag"], o)
        dk, de = torch.autograd.grad((J, A), (s["kappa"], s["emission"]), (s["gJ"], s["gA"]))
        return J.detach(), A.detach(), tot, dk, de
    if do == "ionise":
        t, y, _ = sw.evolve_ionisation(s["dag"], s["emission"], s["params"], 1e30,
                                       neutral=s["neutral"].clone(), max_steps=case["steps"])
        return t, y
    dag = sw.build_dag(s["meshes"], s["dirs"], validate=case["validate"], scheme=case["scheme"])
    if do == "build":
        out = sw.forward(dag, s["kappa"], s["emission"], **o) + (dag.depths(),)
    else:
        J, A, tot, saved = sw.forward(dag, s["kappa"], s["emission"], save_for_adjoint=True, **o)
        dk, de = sw.adjoint(dag, s["kappa"], s["emission"], saved, s["gJ"], s["gA"], **o)
        out = (J, A, tot, dk, de, dag.depths())
    dag.close()
    return out


def _cells(case):
    if case["mesh"] == "lattice":
        return case["n"] ** 3
    M, reps = case["meshes"], case["tx"] * case["ty"] * case["tz"]
    ns = [case["n"] if M == 1 else round(case["n"] * (case["n_hi"] / case["n"]) ** (i / (M - 1))) for i in range(M)]
    if case["mesh"] == "jitter":
        ns = [max(4, round(n ** (1 / 3))) ** 3 for n in ns]
    return sum(ns) * reps


def work(case):
    """Every pass reads the graph once (an 8-byte entry per edge, 12 bytes per task: cell, row and
    outflow weight), and fuses, multiplies and divides once per edge and task; a build reads the
    faces and writes both directions' rows; fields are read and written once."""
    C, D, G = _cells(case), case["D"], case["G"]
    T = C * D
    faces = 6 if case["mesh"] == "lattice" else 15.4
    E = T * (3.0 if case["mesh"] == "lattice" else 3.0 if case["scheme"] == "aligned" else 7.5)
    passes = case["n_scat"] * case["n_pbc"]
    if case["merge"] and case["periodic"] and case["n_scat"] > 1:
        passes = max(case["n_scat"], case["n_pbc"])
    passes *= case["steps"]
    sweep = 12 * T + 8 * E
    b, f = passes * sweep + 16.0 * C * G * case["steps"], passes * G * (2 * E + 4 * T)
    if case["do"] in ("grad", "step"):
        b, f = 2 * b + 8 * T * G * passes, 2 * f + passes * G * 4 * T  # phi kept and read back
    if case["do"] in ("build", "step"):
        b += 45.0 * faces * C + 16 * E + 20 * T
        f += 6.0 * faces * T
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------------- 64-bit answer
class _Graph:
    """Every direction's graph in 64 bits: level by level (tasks, edges out of them), the
    outflow weights, and the periodic edges."""

    def __init__(self, meshes, dirs, case):
        dev = "cuda"
        self.D, eps = len(dirs), 1e-12
        off, ptr, nbr, shift = 0, [], [], []
        for m in meshes:
            fp = m["face_ptr"]
            ptr.append(fp[1:] - fp[:-1])
            nb = m["face_nbr"].long()
            nbr.append(torch.where(nb < 0, -1, nb + off))
            shift.append(torch.zeros_like(nb, dtype=torch.bool) if m["face_shift"] is None else m["face_shift"] != 0)
            off += m["cell_volume"].numel()
        cnt = torch.cat(ptr)
        C = self.C = cnt.numel()
        mf = int(cnt.max())
        pos = torch.arange(mf, device=dev)[None, :] + (torch.cumsum(cnt, 0) - cnt)[:, None]
        ok = torch.arange(mf, device=dev)[None, :] < cnt[:, None]
        pos = torch.where(ok, pos, 0)
        nbr = torch.where(ok, torch.cat(nbr)[pos], -1)
        per = torch.where(ok, torch.cat(shift)[pos], False)
        area = torch.where(ok, torch.cat([m["face_area"] for m in meshes])[pos], 0.0)
        nrm = torch.cat([m["face_normal"].reshape(-1, 3) for m in meshes])[pos] * ok[..., None]
        self.V = torch.cat([m["cell_volume"] for m in meshes])
        dv = torch.as_tensor(np.asarray(dirs), device=dev)

        def out_weights(cells, d):
            """[n, mf] weight of every outflow face of these cells' tasks (0: none)."""
            o = dv[d]
            o = o if o.dim() == 2 else o[None, :]
            n = nrm[cells]
            s = o[:, None, 0] * n[..., 0] + o[:, None, 1] * n[..., 1] + o[:, None, 2] * n[..., 2]
            w = torch.where(s > eps, area[cells] * s, 0.0)
            ap = w.sum(1)
            if case["scheme"] == "aligned":
                best = torch.sort(torch.where(s > eps, s, -1.0), dim=1, descending=True, stable=True)[1][:, :3]
                pick = torch.zeros_like(s).scatter_(1, best, 1.0) * (s > eps)
                w = pick * (ap / pick.sum(1).clamp(min=1))[:, None]
            return w, ap

        T = C * self.D
        self.ap = torch.empty(T, dtype=torch.float64, device=dev)
        self.wall = torch.empty(T, dtype=torch.float64, device=dev)
        need = torch.zeros(T, dtype=torch.int32, device=dev)
        psrc, pdst, pw = [], [], []
        every = torch.arange(C, device=dev)
        for d in range(self.D):
            w, ap = out_weights(every, d)
            self.ap[d * C:(d + 1) * C] = ap
            self.wall[d * C:(d + 1) * C] = torch.where(nbr < 0, w, 0.0).sum(1)
            e = (w > 0) & (nbr >= 0) & ~per
            need[d * C:(d + 1) * C] = torch.bincount(nbr[e], minlength=C).int()
            c, j = torch.nonzero((w > 0) & per, as_tuple=True)
            psrc.append(c + d * C)
            pdst.append(nbr[c, j] + d * C)
            pw.append(w[c, j])
        self.psrc, self.pdst, self.pw = torch.cat(psrc), torch.cat(pdst), torch.cat(pw)
        self.levels = []
        front = torch.nonzero(need == 0)[:, 0]
        while front.numel():
            src, dst, wt = [], [], []
            for part in front.split(1 << 20):
                d, c = part // C, part % C
                w, _ = out_weights(c, d)
                i, j = torch.nonzero((w > 0) & (nbr[c] >= 0) & ~per[c], as_tuple=True)
                src.append(part[i])
                dst.append(d[i] * C + nbr[c[i], j])
                wt.append(w[i, j])
            src, dst, wt = torch.cat(src), torch.cat(dst), torch.cat(wt)
            self.levels.append((front, src, dst, wt))
            need.index_add_(0, dst, torch.full_like(dst, -1, dtype=torch.int32))
            front = torch.unique(dst[need[dst] == 0])


class _Solve(torch.autograd.Function):
    """x of (den - W) x = S, every direction, levels in order."""

    @staticmethod
    def forward(ctx, den, S, g):
        T, x = S.clone(), torch.empty_like(S)
        for t, src, dst, w in g.levels:
            x[t] = T[t] / den[t]
            T.index_add_(0, dst, w[:, None] * x[src])
        ctx.save_for_backward(den, x)
        ctx.g = g
        return x

    @staticmethod
    def backward(ctx, gx):
        den, x = ctx.saved_tensors
        T, lam = gx.clone(), torch.empty_like(gx)
        for t, src, dst, w in reversed(ctx.g.levels):
            T.index_add_(0, src, w[:, None] * lam[dst])
            lam[t] = T[t] / den[t]
        return -lam * x, lam, None


def _transport(g, case, kappa, emission, cells):
    """J, absorbed, totals in 64 bits, differentiable in kappa and emission ([C, G], FP64)."""
    D, C, G = g.D, g.C, kappa.shape[1]
    a = case["albedo"] if case["n_scat"] > 1 else 0.0
    V, ap = g.V[:, None], g.ap[:, None]
    kV = kappa * V
    if case["law"] == "exp":
        tau = (kV.repeat(D, 1) / ap).clamp(max=40.0)
        den = ap * torch.exp(tau)
        r = torch.where(tau > 0, ap * torch.expm1(tau) / kV.repeat(D, 1).clamp(min=1e-300), 1.0)
    else:
        den, r = ap + kV.repeat(D, 1), None
    merged = case["merge"] and case["periodic"] and case["n_scat"] > 1
    seq = [(0, k) for k in range(max(case["n_scat"], case["n_pbc"]))] if merged else \
          [(i, k) for i in range(case["n_scat"]) for k in range(case["n_pbc"])]
    x = j = jprev = None
    inflow = before = torch.zeros((C, G), dtype=torch.float64, device="cuda")
    for i, k in seq:
        if merged or k == 0:
            jprev = j
        S = ((emission + (a * kV * jprev if jprev is not None else 0.0)) / D).repeat(D, 1)
        before, inflow = inflow, torch.zeros_like(inflow)
        if k > 0:
            p = torch.zeros_like(S).index_add(0, g.pdst, g.pw[:, None] * x[g.psrc])
            S, inflow = S + p, p.detach().view(D, C, G).sum(0)
        x = _Solve.apply(den, S, g)
        j = (x if r is None else x * r).view(D, C, G).sum(0)
    absorbed = (1 - a) * kV * j
    with torch.no_grad():
        prev = jprev if jprev is not None else torch.zeros_like(j)
        pout = torch.zeros_like(x).index_add(0, g.psrc, g.pw[:, None] * x[g.psrc]).view(D, C, G).sum(0)
        rel = torch.where(inflow + before > 0, (inflow - before).abs() / (inflow + before).clamp(min=1e-300), 0.0)
        rows, c0 = [], 0
        for n in cells:
            s = slice(c0, c0 + n)
            c0 += n
            per = [emission[s], absorbed[s], (g.wall[:, None] * x).view(D, C, G)[:, s].sum(0), inflow[s], pout[s],
                   a * kV[s] * (prev[s] - j[s])]
            both = (inflow[s] + before[s]).sum(0)
            e = [rel[s].amax(0), torch.where(both > 0, (inflow[s] - before[s]).abs().sum(0) / both.clamp(min=1e-300), 0.0)]
            last = [v if case["periodic"] and (merged or case["n_pbc"] > 1) else torch.zeros_like(v) for v in e]
            rows.append(torch.stack([v.sum(0) for v in per] + last, dim=-1))
    return j / (4 * math.pi), absorbed, torch.stack(rows)


def exact(case, seed):
    passes = case["n_scat"] * case["n_pbc"] * case["steps"]
    if _cells(case) * case["D"] * (1 if case["mesh"] == "lattice" else 4) * case["G"] * min(passes, 4) > 8e8:
        return None
    meshes, dirs, kappa, emission = _inputs(case, seed)
    g = _Graph(meshes, dirs, case)
    cells = [m["cell_volume"].numel() for m in meshes]
    e = emission.double()
    if case["do"] == "ionise":
        p, y = _hii(case, seed)
        V = g.V * p["length_unit"] ** 3
        nH, aB, rate = p["n_H"], p["alpha_B"], p["photon_rate"]
        t = 0.0
        for _ in range(case["steps"]):
            A = _transport(g, case, (nH * p["sigma_H"] * p["length_unit"] * y)[:, None], e, cells)[1][:, 0]
            u = 1 - y
            net = rate * A - aB * nH ** 2 * u * u * V
            lim = torch.where(net > 0, nH * V * y / net, math.inf).min().item()
            dt = min(p["dt_max"], p["courant"] * lim)
            b = u + rate * A * dt / (nH * V)
            y = 1 - (2 * b / (1 + torch.sqrt(1 + 4 * aB * nH * dt * b))).clamp(max=1.0)
            t += dt
        return t, y
    k = kappa.double()
    if case["do"] in ("grad", "step"):
        k.requires_grad_(True)
        e.requires_grad_(True)
        J, A, tot = _transport(g, case, k, e, cells)
        gJ, gA = _loss_grads(case, seed, k.shape[0])
        dk, de = torch.autograd.grad((J, A), (k, e), (gJ.double(), gA.double()))
        return (J.detach(), A.detach(), tot, dk, de) + ((None,) if case["do"] == "step" else ())
    with torch.no_grad():
        J, A, tot = _transport(g, case, k, e, cells)
    return (J, A, tot) + ((None,) if case["do"] == "build" else ())
