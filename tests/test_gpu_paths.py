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
