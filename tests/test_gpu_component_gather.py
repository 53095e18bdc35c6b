"""Operators with three input components, on tiles with elements missing and the most dofs per
thread: vector operators against the scalar one per component, the divergence against the
gradient it is the transpose of."""
import pytest

import synth

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (3, 2, 1), (5, 3, 3)]


@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("kind", ["mass", "diffusion"])
@pytest.mark.parametrize("constrained", [True, False])
def test_vector_equals_components(p, n, kind, constrained):
    import torch
    from paper_1911_09220_amd import pafem as P
    code = P.MASS if kind == "mass" else P.DIFFUSION
    S = P.Space(P.Mesh.from_dict(synth.hex_lattice(n, 0.1, seed=p, rotate_seed=p)), p)
    g = torch.Generator(device="cuda").manual_seed(p)
    qd = S.qdata(code)
    x = torch.randn(3, S.ndofs, dtype=torch.float64, device="cuda", generator=g)
    one = P.Operator(S, code, qd, constrained=constrained)
    want = torch.stack([one.apply(c) for c in x])
    got = P.Operator(S, code, qd, constrained=constrained, vector=True).apply(x.reshape(-1))
    # the same products, summed per dof over at most 8 elements in another order
    assert float((got.reshape(3, -1) - want).norm()) <= 1e-13 * float(want.norm())


@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("n", SIZES)
def test_divergence_is_the_transposed_gradient(p, n):
    import torch
    from paper_1911_09220_amd import pafem as P
    S = P.Space(P.Mesh.from_dict(synth.hex_lattice(n, 0.1, seed=p, rotate_seed=p)), p)
    g = torch.Generator(device="cuda").manual_seed(p)
    # (div u, q) = -(u, grad q) for q = 0 on the boundary
    u = torch.randn(3 * S.ndofs, dtype=torch.float64, device="cuda", generator=g)
    q = torch.randn(S.ndofs, dtype=torch.float64, device="cuda", generator=g)
    q[torch.from_numpy(S.boundary_dofs()).cuda().long()] = 0.0
    D = P.Operator(S, P.DIVERGENCE, S.qdata(P.DIVERGENCE), constrained=False)
    G = P.Operator(S, P.GRADIENT, S.qdata(P.GRADIENT), constrained=False)
    du, gq = D.apply(u), G.apply(q)
    scale = float(du.norm() * q.norm() + gq.norm() * u.norm())
    # both forms integrate polynomials of the reference element exactly (q1d = p + 2 on a
    # trilinear map: degree 2p + 2 per axis at most, 2p + 3 is exact), so they differ by rounding alone
    assert abs(float(du @ q) + float(u @ gq)) <= 1e-11 * max(scale, 1e-300)
