"""H(curl) mass and curl-curl on both sides of the grid size where their kernels load ahead, against
the definite Maxwell kernel with the other coefficient 0."""
import pytest

import synth

pytestmark = pytest.mark.gpu


# 256 tiles of 10 (p = 3) and 7 (p = 4) elements, and the next larger box
@pytest.mark.parametrize("p,n", [(3, (3, 3, 3)), (3, (16, 16, 10)), (3, (16, 16, 11)),
                                 (4, (3, 2, 3)), (4, (16, 16, 7)), (4, (16, 16, 8))])
@pytest.mark.parametrize("kind", ["mass", "curlcurl"])
@pytest.mark.parametrize("constrained", [True, False])
def test_equals_maxwell_part(p, n, kind, constrained):
    import torch
    from paper_1911_09220_amd import pafem as P
    S = P.Space(P.Mesh.from_dict(synth.hex_lattice(n, 0.05, seed=1, rotate_seed=2)), p, family="nd")
    g = torch.Generator(device="cuda").manual_seed(3)
    c = torch.rand(S.nelem * (p + 2) ** 3, dtype=torch.float64, device="cuda", generator=g) + 0.5
    pair = torch.zeros(c.numel(), 2, dtype=torch.float64, device="cuda")
    pair[:, 1 if kind == "mass" else 0] = c
    code = P.HCURL_MASS if kind == "mass" else P.HCURL_CURLCURL
    A = P.Operator(S, code, S.qdata(code, coeff=c), constrained=constrained)
    M = P.Operator(S, P.HCURL_MAXWELL, S.qdata(P.HCURL_MAXWELL, coeff=pair.reshape(-1)),
                   constrained=constrained)
    x = torch.randn(S.ndofs, dtype=torch.float64, device="cuda", generator=g)
    want, got = M.apply(x), A.apply(x)
    # the same products, and per dof the sums of at most 4 elements in another order
    assert float((got - want).norm()) <= 1e-13 * float(want.norm())
