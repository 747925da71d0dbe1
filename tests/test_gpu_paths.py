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


@pytest.mark.parametrize("L,prec", [(16, "fp64"), (72, "fp64"), (72, "mixed"), (96, "fp64"),
                                    (96, "mixed"), (192, "mixed")])
def test_step_at_x_pass_shapes(torch_cuda, L, prec):
    """One step of a few particles from a random field at the edges whose
    forward x pass has its own rows per block and elements per thread (the
    spread boxes folded in it), and the mean mode from its partial sums."""
    torch = torch_cuda
    from paper_1407_5600_amd import Grid, Springs
    say("x pass shape", L, prec)
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
