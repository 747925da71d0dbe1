"""The solve's passes at the sizes whose blocks, elements per thread and cache
hints have rules of their own, against the solve in plain torch in float64."""
import pytest

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-5}
RHO, ETA, DT = 1.3, 0.7, 0.05


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1407_5600_amd  # noqa: F401  (loads the library, fails loudly)
    return torch


def say(*a):
    print("[case]", *a, flush=True)


def plain_solve(torch, v, f, steady):
    """v' of Q (C v + f) mode by mode: C = rho/dt - eta |D|^2 / 2 and Q the
    projection over rho/dt + eta |D|^2 / 2 (steady: over eta |D|^2, no v and no
    mean), D_b = 1 - exp(-2 pi i m_b / L)."""
    L = f.shape[-1]
    dim = (-3, -2, -1)
    m = torch.arange(L, dtype=torch.float64, device="cuda") * (2 * torch.pi / L)
    d = torch.polar(torch.ones_like(m), -m)
    d = 1 - d
    D = (d[None, None, :L // 2 + 1], d[None, :, None], d[:, None, None])
    d2 = sum(x.abs() ** 2 for x in D)
    r = torch.fft.rfftn(f, dim=dim)
    if not steady:
        r += (RHO / DT - 0.5 * ETA * d2) * torch.fft.rfftn(v, dim=dim)
    mean = r[:, 0, 0, 0].clone()
    d2[0, 0, 0] = 1.0
    p = sum(D[b] * r[b] for b in range(3)) / d2
    for b in range(3):
        r[b] = (r[b] - D[b].conj() * p) / (ETA * d2 if steady else RHO / DT + 0.5 * ETA * d2)
    r[:, 0, 0, 0] = 0.0 if steady else mean * DT / RHO
    return torch.fft.irfftn(r, s=(L, L, L), dim=dim)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("mode", ["unsteady", "steady"])
@pytest.mark.parametrize("L", [144, 192, 216, 256, 288, 384, 432])
def test_fluid_solve_in_place_and_not(torch_cuda, L, mode, prec):
    """Every large edge, both flows: into another field, and twice in place
    over the velocity (the second solve reads what the first stored)."""
    torch = torch_cuda
    from paper_1407_5600_amd import Grid
    say("solve", L, mode, prec)
    g = Grid(L, rho=RHO, eta=ETA, dt=DT, precision=prec, mode=mode)
    gen = torch.Generator("cuda").manual_seed(L)
    v, f = (torch.randn(g.field_shape, dtype=torch.float64, device="cuda", generator=gen)
            .to(g.field_dtype) + 0.25 for _ in range(2))
    ref = plain_solve(torch, v.double(), f.double(), mode == "steady")

    def rel(a, b):
        return float(torch.linalg.vector_norm(a.double() - b) / torch.linalg.vector_norm(b))

    out = g.field()
    g.fluid_solve(v, f, out)
    say(f"{rel(out, ref):.2e}")
    assert rel(out, ref) <= TOL[prec]
    w = v.clone()
    g.fluid_solve(w, f, w)
    assert torch.equal(w, out)
    ref = plain_solve(torch, out.double(), f.double(), mode == "steady")
    g.fluid_solve(w, f, w)
    assert rel(w, ref) <= TOL[prec]
