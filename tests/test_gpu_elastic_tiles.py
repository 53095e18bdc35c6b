"""Elasticity on tiles with elements missing and with the most dofs per thread, every order:
the energy of a constant strain, and the constrained apply against the unconstrained one."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("n", [(1, 1, 1), (3, 2, 1), (5, 3, 3)])
@pytest.mark.parametrize("constrained", [True, False])
def test_symmetric_and_exact_energy(p, n, constrained):
    import torch
    from paper_1911_09220_amd import pafem as P
    S = P.Space(P.Mesh.from_dict(synth.hex_lattice(n, 0.1, seed=p, rotate_seed=p)), p)
    npt = S.nelem * (p + 2) ** 3
    lam, mu = 0.7, 1.3
    lm = torch.tensor([lam, mu], dtype=torch.float64, device="cuda").repeat(npt)
    A = P.Operator(S, P.ELASTICITY, S.qdata(P.ELASTICITY, coeff=lm), constrained=False)
    # u = F x has strain sym(F) everywhere: its energy is a volume times a constant, and
    # trilinear geometry represents it exactly
    g = torch.Generator(device="cuda").manual_seed(p)
    F = torch.randn(3, 3, dtype=torch.float64, device="cuda", generator=g)
    X = torch.from_numpy(S.dof_coords()).cuda()
    u = (X @ F.T).T.contiguous().reshape(-1)
    ones = torch.ones(S.ndofs, dtype=torch.float64, device="cuda")
    M = P.Operator(S, P.MASS, S.qdata(P.MASS), constrained=False)
    vol = float(ones @ M.apply(ones))
    E = (F + F.T) / 2
    want = vol * float(lam * torch.trace(F) ** 2 + 2 * mu * (E * E).sum())
    got = float(u @ A.apply(u))
    # sums of at most 1e5 products of rounded factors
    assert abs(got - want) <= 1e-11 * abs(want)
    if not constrained:
        return
    C = P.Operator(S, P.ELASTICITY, S.qdata(P.ELASTICITY, coeff=lm), constrained=True)
    x = torch.randn(3 * S.ndofs, dtype=torch.float64, device="cuda", generator=g)
    b = torch.from_numpy(S.boundary_dofs()).cuda().long()
    ess = torch.cat([b, b + S.ndofs, b + 2 * S.ndofs])
    free = x.clone()
    free[ess] = 0.0
    ref = A.apply(free)
    ref[ess] = x[ess]
    assert float((C.apply(x) - ref).norm()) <= 1e-12 * float(ref.norm())
