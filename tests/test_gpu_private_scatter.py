"""The scatter that stores a tile's private dofs and adds the others, against the
deterministic scatter of the same operator: odd vector addresses, a y that holds rubbish,
essential private dofs, meshes of one tile, several and a ragged last one."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("n", [(1, 1, 1), (3, 2, 5), (9, 8, 7)])
@pytest.mark.parametrize("kind", ["mass", "convection"])
@pytest.mark.parametrize("constrained", [True, False])
@pytest.mark.parametrize("renumber", [True, False])
def test_private_scatter_equals_evec(p, n, kind, constrained, renumber):
    import torch
    from paper_1911_09220_amd import pafem as P
    S = P.Space(P.Mesh.from_dict(synth.hex_lattice(n, 0.1, seed=1, rotate_seed=2)), p, renumber=renumber)
    g = torch.Generator(device="cuda").manual_seed(5)
    q3 = S.nelem * (p + 2) ** 3
    code = P.MASS if kind == "mass" else P.CONVECTION
    coeff = torch.rand(q3 * (1 if kind == "mass" else 3), dtype=torch.float64, device="cuda", generator=g)
    qd = S.qdata(code, coeff=coeff)
    A = P.Operator(S, code, qd, constrained=constrained)
    E = P.Operator(S, code, qd, constrained=constrained, scatter="evec")
    x = torch.randn(S.ndofs + 1, dtype=torch.float64, device="cuda", generator=g)[1:]
    want = E.apply(x)
    y = torch.full((S.ndofs + 3,), float("nan"), dtype=torch.float64, device="cuda")
    for off in (0, 1, 3):
        out = y[off:off + S.ndofs]
        out.fill_(float("nan"))
        A.apply(x, out)
        # each entry sums at most 8 elements' values in another order
        assert float((out - want).abs().max()) <= 16 * 2.0 ** -52 * float(want.abs().max())
    if kind == "mass" and not constrained:
        V = P.Operator(S, code, qd, constrained=constrained, vector=True)
        x3 = torch.randn(3 * S.ndofs, dtype=torch.float64, device="cuda", generator=g)
        y3 = torch.full_like(x3, float("nan"))
        V.apply(x3, y3)
        for c in range(3):
            w = E.apply(x3[c * S.ndofs:(c + 1) * S.ndofs].contiguous())
            assert float((y3[c * S.ndofs:(c + 1) * S.ndofs] - w).abs().max()) <= 16 * 2.0 ** -52 * float(w.abs().max())
