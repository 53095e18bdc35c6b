"""Faces that the velocity is tangential to: the upwind rule takes one side's value there, so a
value that is not finite may cross the face in one direction, never in both."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [1, 2, 4, 6, 8])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_not_finite_crosses_one_way(p, value):
    import torch
    from paper_1911_09220_amd import pafem as P
    # not rotated: beta . N of the tangential faces is 0 exactly (rounding of both signs lets both
    # sides' values through, each at its points)
    mesh = synth.hex_lattice((2, 2, 2), 0.0, seed=1)
    S = P.Space(P.Mesh.from_dict(mesh), p, family="l2")
    beta = torch.tensor([1.0, 0.0, 0.0], dtype=torch.float64, device="cuda")
    A = P.Operator(S, P.DG_CONVECTION, S.qdata(P.DG_CONVECTION, coeff=beta), constrained=False)
    dofs = S.elem_dofs().reshape(8, -1)
    centre = mesh["vertices"][mesh["hex"]].mean(axis=1)
    reached = np.zeros((8, 8), dtype=bool)  # [from, to]
    for e in range(8):
        x = torch.ones(S.ndofs, dtype=torch.float64, device="cuda")
        x[torch.as_tensor(dofs[e], device="cuda").long()] = value
        y = A.apply(x).cpu().numpy()
        reached[e] = [not np.isfinite(y[d]).all() for d in dofs]
    for a in range(8):
        for b in range(8):
            step = centre[b] - centre[a]
            across = np.abs(step) > 0.1
            if a == b or (across.sum() == 1 and step[0] > 0.1):
                assert reached[a, b]  # itself, and downstream
            elif across.sum() > 1 or across[0]:
                assert not reached[a, b]  # no common face, or upstream
            else:
                assert not (reached[a, b] and reached[b, a]), f"{a} and {b}"
