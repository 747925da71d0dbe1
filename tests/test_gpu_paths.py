"""Paths that a call takes by its sizes: each against the oracle, or bit for
bit against the path it replaces, at the sizes on both sides of the rule."""
import numpy as np
import pytest

import oracle
from paper_1407_5600_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-5}


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1407_5600_amd  # noqa: F401  (loads the library, fails loudly)
    return torch


def say(*a):
    print("[case]", *a, flush=True)


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def rel(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return np.linalg.norm((a - b).ravel()) / max(np.linalg.norm(b.ravel()), 1e-300)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("per_box", [0, 5, 2100])
def test_spread_by_component_or_by_box_tile(torch_cuda, prec, per_box):
    """32 boxes of 32^3 have 256 box tiles, spread one component per block;
    33 boxes have 264, spread by whole box tiles.  The sums are in fixed
    point, so the boxes both hold agree bit for bit.  The blobs of a box lie
    in one corner, so most box tiles are empty; 2,100 in one box tile take
    the mixed path's 64-bit sums."""
    torch = torch_cuda
    from paper_1407_5600_amd import Grid
    say("spread split", prec, per_box)
    L = 32
    rng = np.random.default_rng(per_box + 1)
    q = rng.uniform(-1.0, 9.0, size=(33, per_box, 3))
    F = rng.standard_normal((33, per_box, 3))
    out = []
    for nbox in (32, 33):
        g = Grid(L, precision=prec, max_blobs=nbox * max(per_box, 1), nbox=nbox)
        f = torch.full(g.field_shape, 7.0, dtype=g.field_dtype, device="cuda")
        g.spread(dev(torch, q[:nbox].reshape(-1, 3)), dev(torch, F[:nbox].reshape(-1, 3)), f)
        out.append(f.cpu().numpy())
    assert np.array_equal(out[0], out[1][:32])
    if per_box == 0:
        assert not out[1].any()
        return
    for b in (0, 32):
        ref = oracle.spread(oracle.params(L), q[b], F[b])
        assert rel(out[1][b], ref) <= TOL[prec]


@pytest.mark.parametrize("L,prec", [(16, "fp64"), (48, "fp64"), (48, "mixed"), (64, "fp64"),
                                    (64, "mixed"), (72, "fp64"), (72, "mixed"), (96, "fp64"),
                                    (96, "mixed"), (192, "mixed")])
def test_step_at_pass_shapes(torch_cuda, L, prec):
    """One step of a few particles from a random field at the edges whose passes
    have their own rows and columns per block and elements per thread (the
    spread boxes folded in it), and the mean mode from its partial sums."""
    torch = torch_cuda
    from paper_1407_5600_amd import Grid, Springs
    say("pass shapes", L, prec)
    w = inputs.random_suspension(L, L, 5)
    rng = np.random.default_rng(L)
    v0 = rng.standard_normal((3, L, L, L)) + 0.5
    if prec == "mixed":
        v0 = v0.astype(np.float32).astype(np.float64)
    ref = oracle.step(oracle.params(L), w.springs(), w.q, v0, w.Fext, 1)
    g = Grid(L, precision=prec, max_blobs=w.M)
    q, v = dev(torch, w.q), dev(torch, v0).to(g.field_dtype)
    g.step(Springs(w.nb, w.pa, w.pb, w.r0, w.k), q, v, dev(torch, w.Fext))
    r = rel(v.double().cpu().numpy(), ref["v"])
    mean = v.double().mean(dim=(1, 2, 3)).cpu().numpy()
    ref_mean = ref["v"].mean(axis=(1, 2, 3))
    say(f"v {r:.2e} mean {rel(mean, ref_mean):.2e}")
    assert r <= TOL[prec]
    assert rel(mean, ref_mean) <= TOL[prec]


@pytest.mark.parametrize("nb,P", [(1, 681), (1, 683), (13, 51), (13, 52), (13, 53), (64, 10),
                                  (64, 21)])
def test_end_of_call_at_block_edges(torch_cuda, nb, P):
    """A call of eight steps (its own particle order, positions and blob
    velocities copied back, particle means) equals eight calls of one step
    bit for bit, at particle counts around the blocks of the copies (2,048
    float64: 682 particles of one blob, 52 of 13, 10 of 64)."""
    torch = torch_cuda
    from paper_1407_5600_amd import Grid, Springs
    say("end of call", nb, P)
    L = 32
    rng = np.random.default_rng(nb * 1000 + P)
    body = rng.uniform(-1.0, 1.0, size=(nb, 3))
    q0 = (rng.uniform(0, L, size=(P, 1, 3)) + body).reshape(-1, 3)
    pa = np.arange(nb - 1, dtype=np.int32)
    r0 = np.linalg.norm(body[1:] - body[:-1], axis=1)
    F = rng.standard_normal((P, 3))
    out = []
    for calls, steps in ((1, 8), (8, 1)):
        g = Grid(L, precision="mixed", max_blobs=P * nb)
        sp = Springs(nb, pa, pa + 1, r0, 10.0)
        q, v, Fe = dev(torch, q0), g.field(), dev(torch, F)
        u = torch.zeros((P * nb, 3), dtype=torch.float64, device="cuda")
        U0 = torch.zeros((P, 3), dtype=torch.float64, device="cuda")
        for _ in range(calls):
            g.step(sp, q, v, Fe, steps, u_out=u, U0_out=U0)
        out.append([x.cpu().numpy() for x in (q, v, u, U0)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    mean = out[0][2].reshape(P, nb, 3).mean(axis=1)
    # a sum of at most 64 values, each order within n ulps
    assert np.abs(out[0][3] - mean).max() <= nb * 2.3e-16 * np.abs(out[0][2]).max()


@pytest.mark.parametrize("nbox", [200, 260])
def test_diagnostics_in_one_and_two_levels(torch_cuda, nbox):
    """Diagnostics of 200 and 260 boxes of 32^3 (6,400 and 8,320 tile
    partials: one and two levels of the reduction) against torch sums."""
    torch = torch_cuda
    from paper_1407_5600_amd import Grid, Springs
    say("diagnostics", nbox)
    L = 32
    w = inputs.single()
    rng = np.random.default_rng(nbox)
    q = w.q[None] + rng.uniform(0, L, size=(nbox, 1, 3))
    F = rng.standard_normal((nbox, 3))
    g = Grid(L, rho=2.0, max_blobs=w.M * nbox, nbox=nbox)
    v = torch.randn(g.field_shape, dtype=torch.float64, device="cuda",
                    generator=torch.Generator("cuda").manual_seed(nbox)) + 0.25
    diag = torch.zeros(7, dtype=torch.float64, device="cuda")
    g.step(Springs(w.nb, w.pa, w.pb, w.r0, w.k), dev(torch, q.reshape(-1, 3)), v,
           dev(torch, F), diag_out=diag)
    d = diag.cpu().numpy()
    Pi = 2.0 * v.sum(dim=(0, 2, 3, 4)).cpu().numpy()
    assert np.abs(d[:3] - Pi).max() <= 1e-12 * np.abs(Pi).max()
    assert np.abs(d[3:6] - F.sum(0)).max() <= 1e-12 * np.abs(F).sum()
    div = sum(v[:, a] - torch.roll(v[:, a], 1, dims=3 - a) for a in range(3))
    assert d[6] <= 1e-12 and float(div.abs().max()) <= 1e-12


def few_blobs(nb, L, nbox, where, rng):
    """nbox boxes of the most particles of nb blobs that 256 blobs hold, and
    one more at rest without forces: positions far outside the box, across
    its seams, or all within three z planes."""
    P = 256 // nb
    body = rng.uniform(-1.0, 1.0, size=(nb, 3))
    c = rng.uniform(-2 * L, 3 * L, size=(nbox, P + 1, 1, 3))
    if where == "plane":
        body[:, 2] *= 0.2
        c[..., 2] = L + rng.uniform(-0.3, 0.3, size=c.shape[:-1])
    q = c + body
    q[:, :P] += rng.uniform(-0.05, 0.05, size=(nbox, P, nb, 3))
    F = rng.standard_normal((nbox, P + 1, 3))
    F[:, P] = 0.0
    pa = np.arange(nb - 1, dtype=np.int32)
    return P, q, F, (pa, pa + 1, np.linalg.norm(body[1:] - body[:-1], axis=1), 10.0)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nb,L", [(1, 16), (13, 32), (13, 72), (64, 48)])
def test_step_of_few_blobs_per_box(torch_cuda, nb, L, prec):
    """Boxes of at most 256 blobs take their forces in the solve; with one
    more particle, at rest and without forces, they are spread through the
    boxes of tiles.  Both give the same step, in every mode and scheme, with
    and without a force on the fluid.  (The springs of the additional particle
    pull at the midpoint, where the fluid has deformed it: there the step of
    several blobs a particle is held against the oracle.)"""
    torch = torch_cuda
    from paper_1407_5600_amd import Grid, Springs
    nbox = 2
    for i, (where, mode, scheme, forced) in enumerate(
            (w, m, s, f) for w in ("all", "plane") for m in ("unsteady", "steady")
            for s in ("euler", "midpoint") for f in (False, True)):
        say("few blobs", nb, L, prec, where, mode, scheme, forced)
        rng = np.random.default_rng(100 * nb + i)
        P, q0, F0, spr = few_blobs(nb, L, nbox, where, rng)
        vf = rng.standard_normal((2, nbox, 3, L, L, L))
        by_oracle = scheme == "midpoint" and nb > 1
        out = []
        for n in (P,) if by_oracle else (P, P + 1):
            g = Grid(L, precision=prec, mode=mode, scheme=scheme, max_blobs=nbox * n * nb,
                     nbox=nbox)
            q, F = dev(torch, q0[:, :n].reshape(-1, 3)), dev(torch, F0[:, :n].reshape(-1, 3))
            v, f = (dev(torch, x).to(g.field_dtype) for x in vf)
            vs, fs = v.double().cpu().numpy(), f.double().cpu().numpy()
            u = torch.zeros_like(q)
            if forced:
                g.step_forced(Springs(nb, *spr), q, v, f, Fext=F, u_out=u)
            else:
                g.step(Springs(nb, *spr), q, v, F, u_out=u)
            out.append([v.double().cpu().numpy()] +
                       [(x.cpu().numpy().reshape(nbox, n, nb, 3)[:, :P]) for x in (q, u)])
        if by_oracle:
            prm = oracle.params(L, steady=mode == "steady")
            keys = dict(zip(("nb", "pa", "pb", "r0", "k"), (nb,) + spr))
            ref = [oracle.step(prm, keys, q0[b, :P].reshape(-1, 3), vs[b], F0[b, :P],
                               f_fluid=fs[b] if forced else None, scheme=scheme)
                   for b in range(nbox)]
            out.append([np.stack([r[k] for r in ref]) for k in "vqu"])
        for name, a, b in zip(("v", "q", "u"), *out):
            b = b.reshape(a.shape)
            say(name, f"{rel(a, b):.2e}")
            assert rel(a, b) <= TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nb,L", [(1, 16), (13, 72), (64, 48), (13, 192)])
def test_transfer_of_few_blobs_per_box(torch_cuda, nb, L, prec):
    """Spreading, interpolation and its derivative, and (float64) one reverse
    step, at 256 blobs a box and with one more particle of no force and no
    cotangent."""
    torch = torch_cuda
    from paper_1407_5600_amd import Grid, Springs
    for where in ("all", "plane"):
        say("transfer few blobs", nb, L, prec, where)
        rng = np.random.default_rng(100 * nb + L)
        P, q0, F0, spr = few_blobs(nb, L, 1, where, rng)
        W0 = rng.standard_normal(q0.shape)
        W0[:, P] = 0.0
        v0 = rng.standard_normal((3, L, L, L))
        out = []
        for n in (P, P + 1):
            g = Grid(L, precision=prec, max_blobs=n * nb)
            q, W = (dev(torch, x[:, :n].reshape(-1, 3)) for x in (q0, W0))
            v = dev(torch, v0).to(g.field_dtype)
            u, dq = torch.zeros_like(q), torch.zeros_like(q)
            f = g.field()
            g.spread(q, W, f)
            g.interpolate(q, v, u)
            g.interpolate_grad(q, v, W, dq)
            got = [f.double()] + [x[:P * nb] for x in (u, dq)]
            if prec == "fp64":
                qb, vb = W.clone(), v.flip(0).contiguous()
                g.step_adjoint(Springs(nb, *spr), q, v, qb, vb,
                               Fext=dev(torch, F0[0, :n]))
                got += [qb[:P * nb], vb]
            out.append([x.cpu().numpy() for x in got])
        for name, a, b in zip(("f", "u", "dq", "qbar", "vbar"), *out):
            say(name, f"{rel(a, b):.2e}")
            assert rel(a, b) <= TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nb,L,P", [(1, 16, 1), (13, 32, 1), (13, 48, 19), (13, 96, 2)])
def test_steady_steps_of_few_blobs_leave_the_whole_field(torch_cuda, nb, L, P, prec):
    """A steady call of several steps forms the field only on the z planes
    that hold blobs until its last step: positions, velocities and the whole
    field equal those of calls of one step bit for bit, and of the captured
    step, with blobs that cross a seam meanwhile."""
    torch = torch_cuda
    from paper_1407_5600_amd import Grid, Springs
    from paper_1407_5600_amd.binding import step_graph
    rng = np.random.default_rng(nb + L)
    body = rng.uniform(-1.0, 1.0, size=(nb, 3))
    c = rng.uniform(0, L, size=(2, P, 1, 3))
    c[0, 0, 0, 2] = L - 0.02
    q0 = (c + body).reshape(-1, 3)
    F0 = np.abs(rng.standard_normal((2 * P, 3))) * 20.0
    pa = np.arange(nb - 1, dtype=np.int32)
    r0 = np.linalg.norm(body[1:] - body[:-1], axis=1)
    for scheme in ("euler", "midpoint"):
        out = []
        for how in ("one call", "calls", "graph"):
            say("steady few", nb, L, P, prec, scheme, how)
            g = Grid(L, precision=prec, mode="steady", scheme=scheme, dt=0.05,
                     max_blobs=len(q0), nbox=2)
            sp = Springs(nb, pa, pa + 1, r0, 10.0)
            q, F = dev(torch, q0), dev(torch, F0)
            v = torch.full(g.field_shape, 3.0, dtype=g.field_dtype, device="cuda")
            if how == "one call":
                g.step(sp, q, v, F, 7)
            elif how == "calls":
                for _ in range(7):
                    g.step(sp, q, v, F, 1)
            else:
                for n in (1, 4, 2):
                    step_graph([g], [sp], [q], [v], [F], None, n)
            out.append([q.cpu().numpy(), v.cpu().numpy()])
        for other in out[1:]:
            for a, b in zip(out[0], other):
                assert np.array_equal(a, b)


def test_step_noalloc_at_the_scratch_size(torch_cuda):
    """72^3 float64 with 5,915 blobs fills the static scratch but for the
    padding; its step equals a grid's bit for bit."""
    torch = torch_cuda
    from paper_1407_5600_amd import Grid, Springs
    from paper_1407_5600_amd.binding import step_noalloc
    say("noalloc at the scratch size")
    L, P = 72, 455
    w = inputs.random_suspension(L, P, 3)
    sp = Springs(w.nb, w.pa, w.pb, w.r0, w.k)
    g = Grid(L, max_blobs=w.M)
    out = []
    for noalloc in (False, True):
        q, v, F = dev(torch, w.q), g.field(), dev(torch, w.Fext)
        if noalloc:
            step_noalloc(sp, q, v, F, L=L)
        else:
            g.step(sp, q, v, F)
        out.append([q.cpu().numpy(), v.cpu().numpy()])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
