"""Assembly kernels on the apply's tiles against the oracle: quadrature data on every rule
(values and layout, ragged last tiles, both geometries), element diagonals and load vectors
at every order."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _layout(ne, Q, nc):
    """Offset of value (e, c, q) in the tile-interleaved layout, e a device element."""
    nt, qq = max(1, 256 // (Q * Q)), Q * Q
    e, c, q = np.meshgrid(np.arange(ne), np.arange(nc), np.arange(Q ** 3), indexing="ij")
    tile, el, qz, r = e // nt, e % nt, q // qq, q % qq
    if nc in (6, 12):
        return ((tile * (nc // 2) + c // 2) * Q + qz) * nt * qq * 2 + (el * qq + r) * 2 + c % 2
    return ((tile * nc + c) * Q + qz) * nt * qq + el * qq + r


@pytest.mark.parametrize("q1d", range(1, 13))
@pytest.mark.parametrize("geom", [1, 2])
@pytest.mark.parametrize("kind", ["mass", "diffusion", "elasticity", "convection", "gradient"])
def test_qdata_on_every_rule(q1d, geom, kind):
    import torch
    from oracle.forms import _jacobians
    from paper_1911_09220_amd import pafem as P
    mesh = synth.hex_lattice((3, 2, 5), 0.1, seed=1, rotate_seed=2) if geom == 1 else synth.q2_warped_lattice(3)
    S = P.Space(P.Mesh.from_dict(mesh), 2)
    rng = np.random.default_rng(4)
    ne, nq = S.nelem, q1d ** 3
    # one value per element orders the device elements: mass data / (w det J) with coefficient e
    _, w, _, J, det = _jacobians(mesh, q1d)
    Ji = np.linalg.inv(J)
    mass = P.MASS
    ids = np.repeat(np.arange(1, ne + 1, dtype=np.float64), nq)
    raw = S.qdata(mass, q1d=q1d, coeff=torch.as_tensor(ids, device="cuda")).cpu().numpy()[_layout(ne, q1d, 1)][:, 0]
    order = np.empty(ne, dtype=int)
    want = ids.reshape(ne, nq) * w * det
    for k in range(ne):
        order[k] = np.argmin(np.abs(want - raw[k]).max(axis=1))
    assert sorted(order) == list(range(ne))
    assert np.abs(raw - want[order]).max() <= 1e-13 * np.abs(want).max()
    wd = (w * det)
    if kind == "mass":
        return
    if kind == "diffusion":
        c = rng.uniform(0.5, 1.5, size=(ne, nq))
        T = (c * wd)[..., None, None] * np.einsum("eqab,eqcb->eqac", Ji, Ji)
        vals = np.stack([T[..., a, b] for a in range(3) for b in range(a, 3)], axis=1)
        code = P.DIFFUSION
    elif kind == "elasticity":
        c = rng.uniform(0.5, 1.5, size=(ne, nq, 2))
        vals = np.concatenate([np.moveaxis(Ji.reshape(ne, nq, 9), 2, 1), np.moveaxis(c * wd[..., None], 2, 1)], axis=1)
        code = P.ELASTICITY
    elif kind == "convection":
        c = rng.uniform(0.5, 1.5, size=(ne, nq, 3))
        vals = np.moveaxis(wd[..., None] * np.einsum("eqab,eqb->eqa", Ji, c), 2, 1)
        code = P.CONVECTION
    else:
        c = rng.uniform(0.5, 1.5, size=(ne, nq))
        T = (c * wd)[..., None, None] * np.swapaxes(Ji, 2, 3)
        vals = np.moveaxis(T.reshape(ne, nq, 9), 2, 1)
        code = P.GRADIENT
    got = S.qdata(code, q1d=q1d, coeff=torch.as_tensor(c.reshape(-1), device="cuda")).cpu().numpy()
    got = got[_layout(ne, q1d, vals.shape[1])]
    # sums and products of at most 27 nodes' terms and a 3x3 inverse, well conditioned
    assert np.abs(got - vals[order]).max() <= 1e-12 * np.abs(vals).max()


@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("geom", [1, 2])
def test_diagonal_and_load(p, geom):
    import torch
    import oracle
    from oracle import forms
    from paper_1911_09220_amd import pafem as P
    n = 3 if p <= 4 else 2
    mesh = synth.hex_lattice((n, 2, 3), 0.1, seed=1, rotate_seed=2) if geom == 1 else synth.q2_warped_lattice(2)
    S = P.Space(P.Mesh.from_dict(mesh), p)
    q1d = p + 2
    kappa = synth.lognormal_iid(S.nelem, q1d, seed=3)
    kd = torch.as_tensor(kappa.reshape(-1), device="cuda")
    sp = oracle.H1Space(mesh, p)
    X, Xo = S.dof_coords(), sp.dof_coordinates()
    from scipy.spatial import cKDTree
    perm = cKDTree(Xo).query(X)[1]
    for kind, element in ((P.DIFFUSION, forms.element_stiffness), (P.MASS, forms.element_mass)):
        K = oracle.assemble(sp, element(mesh, p, q1d, kappa))
        A = P.Operator(S, kind, S.qdata(kind, coeff=kd), constrained=False)
        want = K.diagonal()[perm]
        assert np.linalg.norm(A.diagonal().cpu().numpy() - want) <= 1e-12 * np.linalg.norm(want)
    f = np.random.default_rng(6).normal(size=kappa.shape)
    want = forms.assemble_vector(sp, forms.element_load(mesh, p, q1d, f))[perm]
    want[S.boundary_dofs()] = 0.0
    got = S.linear_form(P.SOURCE_ARRAY, f_qp=torch.as_tensor(f.reshape(-1), device="cuda")).cpu().numpy()
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
    # the built-in source and the constant, on the fused rule and on the general kernel's
    for src in (P.SOURCE_SINE, P.SOURCE_CONST):
        a = S.linear_form(src, scale=2.0).cpu().numpy()
        b = forms.assemble_vector(sp, forms.element_load(
            mesh, p, q1d, (lambda x: 2.0 * synth.sine_source(x)) if src == P.SOURCE_SINE else (lambda x: np.full(x.shape[:-1], 2.0))))[perm]
        b[S.boundary_dofs()] = 0.0
        assert np.linalg.norm(a - b) <= 1e-12 * np.linalg.norm(b)
        g = S.linear_form(src, q1d=p + 4, scale=2.0).cpu().numpy()
        b = forms.assemble_vector(sp, forms.element_load(
            mesh, p, p + 4, (lambda x: 2.0 * synth.sine_source(x)) if src == P.SOURCE_SINE else (lambda x: np.full(x.shape[:-1], 2.0))))[perm]
        b[S.boundary_dofs()] = 0.0
        assert np.linalg.norm(g - b) <= 1e-12 * np.linalg.norm(b)
