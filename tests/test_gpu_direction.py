"""CG whose applies form their own direction (small grids, zero essential residual): against
plain CG on both sides of the grid size where the direction kernel takes over, stopping inside
a batch, and refinement's buffers carried from a stopped batch to the next step."""
import pytest

import synth

pytestmark = pytest.mark.gpu


def _op(dim, p, n, constrained=True, **kw):
    from paper_1911_09220_amd import pafem as P
    mesh = synth.hex_lattice(n, 0.05, seed=1) if dim == 3 else synth.quad_lattice(n, 0.05, seed=1)
    S = P.Space(P.Mesh.from_dict(mesh), p)
    return P.Operator(S, P.DIFFUSION, S.qdata(P.DIFFUSION), constrained=constrained, **kw)


# 3D: tiles times p + 1 <= 4096 and p <= 7; 2D: 2048 tiles of floor(256 / (p + 2))
@pytest.mark.parametrize("dim,p,n", [(3, p, 2) for p in range(1, 9)] +
                         [(3, 1, 38), (3, 1, 39), (3, 2, 12), (3, 3, 11), (3, 4, 9)] +
                         [(2, p, 5) for p in range(1, 9)] + [(2, 4, 293), (2, 4, 294)])
@pytest.mark.parametrize("constrained", [True, False])
def test_iterates_equal_plain_cg(dim, p, n, constrained):
    import torch
    A = _op(dim, p, n, constrained)
    g = torch.Generator(device="cuda").manual_seed(3)
    ndofs = A.space.ndofs
    # in A's range (the unconstrained A is singular: outside of it CG has no limit and
    # amplifies rounding), 0 on the essential dofs
    b = A.apply(torch.randn(ndofs, dtype=torch.float64, device="cuda", generator=g))
    if constrained:
        b[torch.from_numpy(A.space.boundary_dofs()).cuda().long()] = 0.0
    diag = A.diagonal()
    got, info = A.pcg(b, diag=diag, rel_tol=0.0, max_iter=7, check_every=4)
    ref, r = torch.zeros_like(b), b.clone()
    z = r / diag
    d, rz, hist = z.clone(), r @ z, [1.0]
    for _ in range(info["iters"]):
        if float(rz) == 0.0:  # one free dof: solved exactly
            break
        q = A.apply(d)
        alpha = rz / (d @ q)
        ref += alpha * d
        r -= alpha * q
        z = r / diag
        rz, old = r @ z, rz
        d = z + (rz / old) * d
        hist.append(float(r.norm() / b.norm()))
    assert info["iters"] == 7 or info["rel_res"] < 1e-14
    # seven iterations of FP64 sums of at most 1.4e6 terms: 7 * 1.4e6 * 2^-53 ~ 1e-9
    assert float((got - ref).norm() / ref.norm()) < 2e-9
    assert max(abs(a - c) for a, c in zip(info["history"], hist)) < 2e-9


@pytest.mark.parametrize("dim,p,n", [(3, 2, 8), (3, 6, 4), (2, 4, 24)])
@pytest.mark.parametrize("check", [2, 7, 50])
def test_stops_inside_a_batch(dim, p, n, check):
    A = _op(dim, p, n)
    b, diag = A.space.linear_form(), A.diagonal()
    x, info = A.pcg(b, diag=diag, rel_tol=1e-8, check_every=check)
    xe, ie = A.pcg(b, diag=diag, rel_tol=1e-8, check_every=1)  # every direction on its own
    assert info["converged"] and abs(info["iters"] - ie["iters"]) <= 1
    assert info["rel_res"] <= 1e-8 and len(info["history"]) == info["iters"] + 1
    # the recurrence's residual and the true one part by rounding alone
    assert info["true_rel_res"] < 1.01e-8
    # both are within cond(A) rel_tol of the solution, cond < 1e5
    assert float((x - xe).norm() / xe.norm()) < 2e-3


@pytest.mark.parametrize("p,n", [(1, 12), (3, 6), (6, 5), (8, 3)])
@pytest.mark.parametrize("check", [1, 5, 8])
@pytest.mark.parametrize("keep", [True, False])
def test_refinement_buffers(p, n, check, keep):
    from paper_1911_09220_amd import pafem as P
    out = []
    for scatter in ("atomic", "evec"):
        A = _op(3, p, n, scatter=scatter)
        S = A.space
        L = P.Operator(S, P.DIFFUSION, P.lowered_qdata(S.qdata(P.DIFFUSION), P.F32),
                       qdata_dtype=P.F32, scatter=scatter)
        out.append(A.ir_solve(L, S.linear_form(), rel_tol=1e-10, check_every=check,
                              keep_direction=keep)[1])
    assert out[0]["converged"] and out[0]["rel_res"] <= 1e-10
    # a direction or product from the wrong buffer costs conjugacy, and with it iterations
    assert abs(out[0]["outer"] - out[1]["outer"]) <= 1
    assert abs(out[0]["inner_total"] - out[1]["inner_total"]) <= 2 + out[1]["inner_total"] // 10
