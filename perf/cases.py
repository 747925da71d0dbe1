"""Workloads that programs built on this package run, at the sizes of its
configurations, tests and benchmark, for timing and for comparing outputs.

Every case is a dict of plain values with a "kind":

  step     ``Grid.step`` on one box: P icosahedral particles of 13 blobs, from
           one particle to a dense suspension, one call of `steps` steps
           returning the positions, the field, the particle velocities and
           the diagnostics; float64 or mixed fields, first-order or midpoint
           scheme.
  sweep    ``step_graph`` on several batch grids (one per box edge), two
           particles per box pulled apart in steady Stokes flow: the
           pair-mobility sweeps.
  forced   ``Grid.step_forced`` on a batch of suspensions driven by a shear
           force density in steady Stokes flow: the viscosity measurement.
  diff     loss and gradients of a differentiable trajectory
           (``autodiff.trajectory``) with respect to the initial field, blob
           forces, stiffness and particle radius: forward, recomputation and reverse steps.
  blobs    ``Grid.spread`` and ``Grid.interpolate`` of free blobs, the two
           transfer operators on their own.
  solve    ``Grid.fluid_solve`` of a given velocity and force density.

``exact`` repeats a case in plain torch in float64: per-blob kernel sums by
index, ``torch.fft`` for the solve, autograd for the gradients.
"""
import math

import torch

from paper_1407_5600_amd import Grid, Springs, inputs
from paper_1407_5600_amd.autodiff import particle_means, place_template, trajectory
from paper_1407_5600_amd.binding import step_graph

# Edges with kernels (2^a 3^b, multiples of 8) that the cases use.
EDGES = (16, 24, 32, 48, 64, 72, 96, 128, 144, 192, 216, 256)
NB = 13
STIFFNESS = 100.0


def listed():
    return [
        # an interactive or coupled program: one particle, one step per call,
        # its velocity and the diagnostics read after each
        dict(name="single_32", kind="step", L=32, P=1, precision="fp64", steps=1,
             zero_mean=False, scheme="euler"),
        # a moderate suspension stepped one call at a time, looked at after
        # every step; an edge with a factor of three
        dict(name="step_96", kind="step", L=96, P=7737, precision="fp64", steps=1,
             zero_mean=False, scheme="euler"),
        # the benchmark's dense suspension (128^3, volume fraction 0.3)
        dict(name="dense_128_mixed", kind="step", L=128, P=36669, precision="mixed", steps=20,
             zero_mean=False, scheme="euler"),
        # the same in float64
        dict(name="dense_128_fp64", kind="step", L=128, P=36669, precision="fp64", steps=20,
             zero_mean=False, scheme="euler"),
        # the benchmark's large suspension (256^3, volume fraction 0.4)
        dict(name="large_256_mixed", kind="step", L=256, P=391139, precision="mixed", steps=8,
             zero_mean=False, scheme="euler"),
        # a ragged edge, no net flow (the periodic-array setting)
        dict(name="array_144_mixed", kind="step", L=144, P=43507, precision="mixed", steps=10,
             zero_mean=True, scheme="euler"),
        # the second-order scheme on a small dense box
        dict(name="midpoint_64_fp64", kind="step", L=64, P=4583, precision="fp64", steps=10,
             zero_mean=False, scheme="midpoint"),
        # the pair-mobility sweep: four box sizes, a HIP graph of one step
        dict(name="pair_sweep", kind="sweep", boxes=32, precision="mixed", steps=50,
             small=24, large=64),
        # the viscosity measurement: sheared 32^3 suspensions of volume fraction 0.15
        dict(name="viscosity", kind="forced", L=32, boxes=16, P=276, precision="fp64", steps=20),
        # the differentiation case: 64^3, 16 particles, 100 steps
        dict(name="gradient_64", kind="diff", L=64, P=16, steps=100, every=10),
        # the transfer operators on free blobs, an odd number of them
        dict(name="transfer_72", kind="blobs", L=72, M=50001, precision="fp64"),
        # the fluid solve alone
        dict(name="solve_192", kind="solve", L=192, precision="fp64", mode="unsteady"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _edge(rng, lo, hi):
    x = rng.uniform(math.log(lo), math.log(hi))
    return min((e for e in EDGES if lo <= e <= hi), key=lambda e: abs(math.log(e) - x))


def _most_particles(L, phi):
    return max(1, inputs.particles_for_fraction(L, phi))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "step", "sweep", "forced", "diff",
                       "blobs", "solve"])
    precision = rng.choice(["fp64", "mixed"])
    if kind == "step":
        L = _edge(rng, 16, 256)
        # a few particles, or a suspension of volume fraction up to 0.4
        P = (_log_int(rng, 1, 64) if rng.random() < 0.3
             else _most_particles(L, rng.uniform(0.02, 0.4)))
        P = min(P, _most_particles(L, 0.4))
        cap = 8 * 256 ** 3 // (L ** 3 * (2 if precision == "fp64" else 1))
        return dict(kind=kind, L=L, P=P, precision=precision,
                    steps=_log_int(rng, 1, max(1, min(20, cap))),
                    zero_mean=rng.random() < 0.3,
                    scheme="midpoint" if rng.random() < 0.2 else "euler")
    if kind == "sweep":
        small = rng.choice([16, 24, 32])
        return dict(kind=kind, boxes=rng.randint(3, 31), precision=precision,
                    steps=rng.randint(10, 50), small=small,
                    large=rng.choice([e for e in (32, 48, 64) if e > small]))
    if kind == "forced":
        L = rng.choice([24, 32, 48])
        return dict(kind=kind, L=L, boxes=rng.randint(2, 16),
                    P=_most_particles(L, rng.uniform(0.03, 0.2)), precision=precision,
                    steps=_log_int(rng, 1, 20))
    if kind == "diff":
        L = rng.choice([24, 32, 48, 64])
        return dict(kind=kind, L=L, P=rng.randint(1, 24), steps=rng.randint(5, 60),
                    every=rng.choice([5, 10]))
    if kind == "blobs":
        L = _edge(rng, 24, 192)
        return dict(kind=kind, L=L, M=_log_int(rng, 11, L ** 3 // 6), precision=precision)
    return dict(kind=kind, L=_edge(rng, 16, 256), precision=precision,
                mode=rng.choice(["unsteady", "steady"]))


# ---- Inputs -----------------------------------------------------------------
def _template(a=1.0):
    tmpl = inputs.icosahedron_template(a)
    pa, pb, r0 = inputs.pair_table(tmpl)
    return tmpl, pa, pb, r0


def _rotations(gen, n):
    """n uniformly random rotation matrices (normalised Gaussian quaternions)."""
    qt = torch.randn((n, 4), dtype=torch.float64, generator=gen)
    w, x, y, z = (qt / qt.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                        2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                        2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)],
                       1).view(n, 3, 3)


def _centres(gen, L, n):
    """n centres that keep apart: a random subset of a cubic lattice, each
    displaced within its cell as far as particles of diameter 3.2 allow, the
    whole shifted at random, in random order."""
    m = 1
    while m ** 3 < n:
        m += 1
    pick = torch.randperm(m ** 3, generator=gen)[:n]
    c = torch.stack([pick % m, (pick // m) % m, pick // (m * m)], 1).double() + 0.5
    slack = max(0.5 * (L / m - 2 * inputs.EFFECTIVE_RADIUS), 0.0)
    jit = 2 * torch.rand((n, 3), dtype=torch.float64, generator=gen) - 1
    shift = L * torch.rand((1, 3), dtype=torch.float64, generator=gen)
    return (c * (L / m) + slack * jit + shift) % L


def _particles(gen, L, n):
    """Blobs of n randomly oriented particles (n * 13, 3), on the host."""
    tmpl = torch.from_numpy(_template()[0])
    body = torch.matmul(_rotations(gen, n), tmpl.T).transpose(1, 2)
    return (_centres(gen, L, n)[:, None, :] + body).reshape(-1, 3).contiguous()


def _flow(gen, L, amplitude=0.02):
    """A smooth periodic velocity field (3, L, L, L) in float64: per component
    four Fourier modes of wave numbers up to 3, on the GPU."""
    x = torch.arange(L, dtype=torch.float64, device="cuda") * (2 * math.pi / L)
    v = torch.zeros((3, L, L, L), dtype=torch.float64, device="cuda")
    for c in range(3):
        for _ in range(4):
            k = torch.randint(-3, 4, (3,), generator=gen).tolist()
            ph = 2 * math.pi * torch.rand(1, dtype=torch.float64, generator=gen).item()
            a = amplitude * torch.randn(1, dtype=torch.float64, generator=gen).item()
            v[c] += a * torch.sin(k[2] * x[:, None, None] + k[1] * x[None, :, None]
                                  + k[0] * x[None, None, :] + ph)
    return v


def _shear(L, boxes, f0=1e-5):
    """The force density f0 sin(2 pi y / L) along x of every box."""
    y = torch.arange(L, dtype=torch.float64, device="cuda") * (2 * math.pi / L)
    f = torch.zeros((boxes, 3, L, L, L), dtype=torch.float64, device="cuda")
    f[:, 0] = f0 * torch.sin(y)[None, None, :, None]
    return f


def _edges(case):
    return [e for e in (16, 24, 32, 48, 64) if case["small"] <= e <= case["large"]]


def _data(case, seed):
    """The case's inputs on the GPU in float64, fields rounded to the case's
    field type: what both the framework and `exact` start from."""
    gen = torch.Generator().manual_seed(int(seed))
    ft = torch.float32 if case.get("precision") == "mixed" else torch.float64
    kind = case["kind"]
    if kind == "step":
        q = _particles(gen, case["L"], case["P"])
        F = torch.randn((case["P"], 3), dtype=torch.float64, generator=gen)
        return dict(q=q.cuda(), F=F.cuda(), v=_flow(gen, case["L"]).to(ft))
    if kind == "sweep":
        out = []
        tmpl = torch.from_numpy(_template()[0])
        for L in _edges(case):
            B = case["boxes"]
            sep = 2 + 4 * torch.rand(B, dtype=torch.float64, generator=gen)
            mid = L / 2 + torch.rand((B, 3), dtype=torch.float64, generator=gen) - 0.5
            c = torch.stack([mid, mid], 1)
            c[:, 0, 0] -= sep / 2
            c[:, 1, 0] += sep / 2
            body = torch.matmul(_rotations(gen, B), tmpl.T).transpose(1, 2)
            q = (c[:, :, None, :] + body[:, None]).reshape(-1, 3).contiguous()
            F = torch.zeros((B, 2, 3), dtype=torch.float64)
            # as the sweep pulls in float64; weakly in mixed precision, as the
            # other Stokes-limit measurements do
            pull = 1.0 if ft == torch.float64 else 0.01
            F[:, 0, 0], F[:, 1, 0] = pull, -pull
            out.append(dict(q=q.cuda(), F=F.reshape(-1, 3).cuda()))
        return out
    if kind == "forced":
        L, B = case["L"], case["boxes"]
        q = torch.cat([_particles(gen, L, case["P"]) for _ in range(B)])
        return dict(q=q.cuda(), f=_shear(L, B).to(ft))
    if kind == "diff":
        P, L = case["P"], case["L"]
        F = torch.randn((P, 3), dtype=torch.float64, generator=gen)
        return dict(c=_centres(gen, L, P).cuda(), R=_rotations(gen, P).cuda(),
                    G=(F / NB).repeat_interleave(NB, 0).cuda(),
                    V=0.1 * torch.randn((P, 3), dtype=torch.float64, generator=gen).cuda())
    dg = torch.Generator(device="cuda").manual_seed(int(seed))

    def noise(*shape):
        return torch.randn(shape, dtype=torch.float64, device="cuda", generator=dg)

    L = case["L"]
    if kind == "blobs":
        q = L * (3 * torch.rand((case["M"], 3), dtype=torch.float64, device="cuda",
                                generator=dg) - 1)
        return dict(q=q, F=noise(case["M"], 3), v=noise(3, L, L, L).to(ft))
    return dict(v=noise(3, L, L, L).to(ft), f=noise(3, L, L, L).to(ft))


def prepare(case, seed):
    d = _data(case, seed)
    kind = case["kind"]
    tmpl, pa, pb, r0 = _template()
    st = dict(case=case)
    if kind == "step":
        st.update(d, grid=Grid(case["L"], dt=0.01, precision=case["precision"],
                               zero_mean=case["zero_mean"], scheme=case["scheme"],
                               max_blobs=d["q"].shape[0]),
                  springs=Springs(NB, pa, pb, r0, STIFFNESS),
                  U0=torch.zeros((case["P"], 3), dtype=torch.float64, device="cuda"),
                  diag=torch.zeros(7, dtype=torch.float64, device="cuda"))
    elif kind == "sweep":
        sp = Springs(NB, pa, pb, r0, STIFFNESS)
        gs = [Grid(L, dt=0.05, precision=case["precision"], mode="steady", zero_mean=True,
                   max_blobs=x["q"].shape[0], nbox=case["boxes"])
              for L, x in zip(_edges(case), d)]
        st.update(grids=gs, springs=[sp] * len(gs), q=[x["q"] for x in d],
                  F=[x["F"] for x in d], v=[g.field() for g in gs])
    elif kind == "forced":
        g = Grid(case["L"], dt=0.02, precision=case["precision"], mode="steady",
                 zero_mean=True, max_blobs=d["q"].shape[0], nbox=case["boxes"])
        st.update(d, grid=g, v=g.field(), springs=Springs(NB, pa, pb, r0, STIFFNESS))
    elif kind == "diff":
        L = case["L"]
        st.update(d, grid=Grid(L, dt=0.01, max_blobs=case["P"] * NB), pa=pa, pb=pb,
                  unit=torch.from_numpy(tmpl).cuda(), r0=torch.from_numpy(r0).cuda(),
                  v0=torch.zeros((3, L, L, L), dtype=torch.float64, device="cuda"))
    elif kind == "blobs":
        st.update(d, grid=Grid(case["L"], precision=case["precision"], max_blobs=case["M"]))
    else:
        st.update(d, grid=Grid(case["L"], dt=0.01, precision=case["precision"],
                               mode=case["mode"]))
    return st


def _leaf(x):
    return torch.tensor(x, dtype=torch.float64, device="cuda", requires_grad=True)


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "step":
        st["grid"].step(st["springs"], st["q"], st["v"], st["F"], case["steps"],
                        U0_out=st["U0"], diag_out=st["diag"])
        if case["precision"] == "mixed":
            # kept with the accuracy of a mixed step's fields
            return st["q"], st["v"], st["U0"].float(), st["diag"].float()
        return st["q"], st["v"], st["U0"], st["diag"]
    if kind == "sweep":
        step_graph(st["grids"], st["springs"], st["q"], st["v"], st["F"], None, case["steps"])
        return st["q"], st["v"]
    if kind == "forced":
        st["grid"].step_forced(st["springs"], st["q"], st["v"], st["f"], nsteps=case["steps"])
        return st["q"], st["v"]
    if kind == "diff":
        a, k = _leaf(1.0), _leaf(STIFFNESS)
        G = st["G"].detach().requires_grad_(True)
        v0 = st["v0"].detach().requires_grad_(True)
        q0 = place_template(st["c"], st["R"], st["unit"], a)
        u = trajectory(st["grid"], NB, st["pa"], st["pb"], q0, v0, G, k, a * st["r0"],
                       case["steps"], case["every"])
        loss = ((particle_means(u, NB) - st["V"]) ** 2).sum()
        loss.backward()
        return loss.detach(), u.detach(), v0.grad, G.grad, k.grad, a.grad
    if kind == "blobs":
        f = st["grid"].spread(st["q"], st["F"])
        u = st["grid"].interpolate(st["q"], st["v"])
        return f, u.float() if case["precision"] == "mixed" else u
    return st["grid"].fluid_solve(st["v"], st["f"])


# ---- What a pass cannot do without --------------------------------------------
def _step_work(L, boxes, P, s, steady=False, fields=1):
    """One step: the field read (unless steady) and written, positions read
    and written, forces read; two real-to-complex 3-D transforms of three
    components, the solve, 27 nodes per component each way and 78 springs."""
    N = boxes * L ** 3
    M = NB * P
    by = (fields + (0 if steady else 1)) * 3 * N * s + 48 * M + 24 * P
    fl = 2 * 3 * 2.5 * N * 3 * math.log2(L) + 40 * N + M * (2 * 81 * 4 + 12 * 20)
    return by, fl


def work(case):
    kind = case["kind"]
    s = 4 if case.get("precision") == "mixed" else 8
    if kind == "step":
        by, fl = _step_work(case["L"], 1, case["P"], s)
        n = case["steps"]
    elif kind == "sweep":
        each = [_step_work(L, case["boxes"], 2 * case["boxes"], s, True) for L in _edges(case)]
        by, fl, n = sum(b for b, _ in each), sum(f for _, f in each), case["steps"]
    elif kind == "forced":
        by, fl = _step_work(case["L"], case["boxes"], case["P"] * case["boxes"], s, True, 2)
        n = case["steps"]
    elif kind == "diff":
        # forward, and the reverse step with its two fields; the states in
        # between are recomputed
        by, fl = _step_work(case["L"], 1, case["P"], s)
        by, fl, n = 4 * by, 3 * fl, case["steps"]
    elif kind == "blobs":
        by = 2 * 3 * case["L"] ** 3 * s + 4 * 24 * case["M"]
        fl, n = 2 * 81 * 4 * case["M"], 1
    else:
        N = case["L"] ** 3
        by = (3 if case["mode"] == "unsteady" else 2) * 3 * N * s
        fl, n = 2 * 3 * 2.5 * N * 3 * math.log2(case["L"]) + 40 * N, 1
    return {"bytes": by * n, "flops": fl * n}


# ---- The same in plain torch, float64 -----------------------------------------
def _nodes(q, L, a):
    """Per blob and axis: the three node indices of component a's node set
    (M, 3 nodes) and their kernel weights."""
    idx, wgt = [], []
    for b in range(3):
        x = q[:, b] - (0.5 if a == b else 0.0)
        i0 = torch.floor(x + 0.5).detach()
        t = x - i0
        s = torch.sqrt(1 - 3 * t * t)
        wgt.append(torch.stack([(2 - 3 * t - s) / 6, (1 + s) / 3, (2 + 3 * t - s) / 6], 1))
        i = i0.long()
        idx.append(torch.stack([i - 1, i, i + 1], 1) % L)
    return idx, wgt


def _stencil(q, box, L, a):
    """Linear node indices (M, 27) into component a of the fields of all
    boxes, viewed (boxes, L^3), and their weights."""
    (ix, iy, iz), (wx, wy, wz) = _nodes(q, L, a)
    lin = ((box[:, None, None, None] * L + iz[:, :, None, None]) * L
           + iy[:, None, :, None]) * L + ix[:, None, None, :]
    w = wz[:, :, None, None] * wy[:, None, :, None] * wx[:, None, None, :]
    return lin.reshape(-1, 27), w.reshape(-1, 27)


CHUNK = 1 << 20


def _x_spread(q, F, boxes, L):
    M = q.shape[0]
    box = torch.arange(M, device=q.device) // max(M // boxes, 1)
    comps = []
    for a in range(3):
        f = torch.zeros(boxes * L ** 3, dtype=torch.float64, device=q.device)
        for c in range(0, M, CHUNK):
            lin, w = _stencil(q[c:c + CHUNK], box[c:c + CHUNK], L, a)
            f = f.index_add(0, lin.reshape(-1), (w * F[c:c + CHUNK, a, None]).reshape(-1))
        comps.append(f.view(boxes, L, L, L))
    return torch.stack(comps, 1)


def _x_interp(q, v, boxes, L):
    M = q.shape[0]
    box = torch.arange(M, device=q.device) // max(M // boxes, 1)
    out = []
    for a in range(3):
        va = v[:, a].reshape(-1)
        part = []
        for c in range(0, M, CHUNK):
            lin, w = _stencil(q[c:c + CHUNK], box[c:c + CHUNK], L, a)
            part.append((w * va[lin]).sum(1))
        out.append(torch.cat(part))
    return torch.stack(out, 1)


def _x_solve(v, f, L, dt, steady, zero_mean):
    """Crank-Nicolson (rho = eta = 1) or steady Stokes step of the fields
    (boxes, 3, L, L, L) with the projection on discretely solenoidal ones."""
    k = torch.arange(L, dtype=torch.float64, device=f.device) * (2 * math.pi / L)
    kr = k[: L // 2 + 1]
    d2 = ((2 - 2 * torch.cos(k))[:, None, None] + (2 - 2 * torch.cos(k))[None, :, None]
          + (2 - 2 * torch.cos(kr))[None, None, :])

    def sym(x):
        return torch.complex(1 - torch.cos(x), torch.sin(x))

    D = (sym(kr)[None, None, :], sym(k)[None, :, None], sym(k)[:, None, None])
    fh = torch.fft.rfftn(f, dim=(-3, -2, -1))
    d2s = d2.clone()
    d2s[0, 0, 0] = 1.0
    if steady:
        r, den = fh, d2s
    else:
        r = (1 / dt - 0.5 * d2) * torch.fft.rfftn(v, dim=(-3, -2, -1)) + fh
        den = 1 / dt + 0.5 * d2
    div = sum(D[a] * r[:, a] for a in range(3)) / d2s
    o = torch.stack([(r[:, a] - D[a].conj() * div) / den for a in range(3)], 1)
    if steady or zero_mean:  # else the mean mode evolves: D = 0 leaves it unprojected
        keep = torch.ones_like(d2)
        keep[0, 0, 0] = 0.0
        o = o * keep
    return torch.fft.irfftn(o, s=(L, L, L), dim=(-3, -2, -1))


def _x_springs(q, F, Gblob, k, r0, pa, pb):
    x = q.view(-1, NB, 3)
    d = x[:, pb] - x[:, pa]
    ln = d.norm(dim=2, keepdim=True)
    f = k * (ln - r0[None, :, None]) * d / ln
    out = torch.zeros_like(x).index_add(1, pa, f).index_add(1, pb, -f)
    if F is not None:
        out = out + F[:, None, :] / NB
    out = out.reshape(-1, 3)
    return out if Gblob is None else out + Gblob


def _x_table():
    _, pa, pb, r0 = _template()
    return (torch.from_numpy(pa).long().cuda(), torch.from_numpy(pb).long().cuda(),
            torch.from_numpy(r0).cuda())


def _x_steps(q, v, boxes, L, dt, steps, steady, zero_mean, F=None, f_fluid=None,
             scheme="euler"):
    pa, pb, r0 = _x_table()

    def solve(x):
        b = _x_springs(x, F, None, STIFFNESS, r0, pa, pb)
        f = _x_spread(x, b, boxes, L)
        return b, _x_solve(v, f if f_fluid is None else f + f_fluid, L, dt, steady, zero_mean)

    for _ in range(steps):
        if scheme == "euler":
            b, v = solve(q)
            u = _x_interp(q, v, boxes, L)
        else:
            qs = q + 0.5 * dt * _x_interp(q, v, boxes, L)
            old = v
            b, v = solve(qs)
            u = _x_interp(qs, 0.5 * (old + v), boxes, L)
        q = q + dt * u
    div = sum(v[:, a] - torch.roll(v[:, a], 1, dims=3 - a) for a in range(3))
    diag = torch.cat([v.sum(dim=(0, 2, 3, 4)), b.sum(0), div.abs().max().view(1)])
    return q, v, u, diag


def exact(case, seed):
    d = _data(case, seed)
    kind = case["kind"]
    if kind == "step":
        L = case["L"]
        q, v, u, diag = _x_steps(d["q"], d["v"].double()[None], 1, L, 0.01, case["steps"],
                                 False, case["zero_mean"], d["F"], scheme=case["scheme"])
        return q, v[0], u.view(-1, NB, 3).mean(1), diag
    if kind == "sweep":
        qs, vs = [], []
        for L, x in zip(_edges(case), d):
            q, v, _, _ = _x_steps(x["q"], None, case["boxes"], L, 0.05, case["steps"], True,
                                  True, x["F"])
            qs.append(q)
            vs.append(v)
        return qs, vs
    if kind == "forced":
        q, v, _, _ = _x_steps(d["q"], None, case["boxes"], case["L"], 0.02, case["steps"],
                              True, True, None, d["f"].double())
        return q, v
    if kind == "diff":
        L, dt = case["L"], 0.01
        pa, pb, r0u = _x_table()
        a, k = _leaf(1.0), _leaf(STIFFNESS)
        G = d["G"].requires_grad_(True)
        body = torch.matmul(d["R"], torch.from_numpy(_template()[0]).cuda().T).transpose(1, 2)
        q = (d["c"][:, None, :] + a * body).reshape(-1, 3)
        v0 = torch.zeros((3, L, L, L), dtype=torch.float64, device="cuda", requires_grad=True)
        v = v0[None]
        for _ in range(case["steps"]):
            b = _x_springs(q, None, G, k, a * r0u, pa, pb)
            v = _x_solve(v, _x_spread(q, b, 1, L), L, dt, False, False)
            u = _x_interp(q, v, 1, L)
            q = q + dt * u
        loss = ((u.view(-1, NB, 3).mean(1) - d["V"]) ** 2).sum()
        loss.backward()
        return loss.detach(), u.detach(), v0.grad, G.grad, k.grad, a.grad
    if kind == "blobs":
        L = case["L"]
        return (_x_spread(d["q"], d["F"], 1, L)[0],
                _x_interp(d["q"], d["v"].double()[None], 1, L))
    v = _x_solve(d["v"].double()[None], d["f"].double()[None], case["L"], 0.01,
                 case["mode"] == "steady", False)
    return v[0]
