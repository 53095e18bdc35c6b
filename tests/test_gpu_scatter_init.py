"""The start of the atomic scatter (y = x on essential dofs, 0 elsewhere): counts of every remainder,
vectors with and without the alignment of its 16-byte stores, one and three components."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(1, 1, 1), (1, 2, 2), (2, 2, 2), (2, 2, 4), (9, 10, 10), (10, 10, 10)])
@pytest.mark.parametrize("shift", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("kind", ["f64", "f32", "vector"])
def test_alignment_and_remainders(n, shift, kind):
    import torch
    from paper_1911_09220_amd import pafem as P
    S = P.Space(P.Mesh.from_dict(synth.hex_lattice(n, 0.1, seed=1)), 1)
    qd = S.qdata(P.DIFFUSION)
    dt = torch.float32 if kind == "f32" else torch.float64
    if kind == "f32":
        A = P.Operator(S, P.DIFFUSION, P.lowered_qdata(qd, P.F32), qdata_dtype=P.F32)
    else:
        A = P.Operator(S, P.DIFFUSION, qd, vector=kind == "vector")
    nc = 3 if kind == "vector" else 1
    N = nc * S.ndofs
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn(N, dtype=dt, device="cuda", generator=g)
    want = A.apply(x)
    bufs = [torch.full((N + 9,), float("nan"), dtype=dt, device="cuda") for _ in range(2)]
    xs, ys = bufs[0][shift[0]:shift[0] + N], bufs[1][shift[1]:shift[1] + N]
    xs.copy_(x)
    A.apply(xs, ys)
    ess = torch.from_numpy(S.boundary_dofs()).cuda().long()
    for c in range(nc):
        assert torch.equal(ys[ess + c * S.ndofs], x[ess + c * S.ndofs])
    # the same products, summed per dof over at most 8 elements in another order
    assert float((ys - want).norm()) <= (1e-5 if kind == "f32" else 1e-13) * float(want.norm())
    rest = torch.cat([bufs[1][:shift[1]], bufs[1][shift[1] + N:]])
    assert bool(rest.isnan().all())  # nothing outside the vector


@pytest.mark.parametrize("n", [(1, 1, 1), (1, 2, 2), (2, 2, 2), (9, 10, 10)])
@pytest.mark.parametrize("shift", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("kind", ["gradient", "divergence", "vector"])
def test_without_constraints(n, shift, kind):
    """One run of zeros over all components, whatever their stride."""
    import torch
    from paper_1911_09220_amd import pafem as P
    S = P.Space(P.Mesh.from_dict(synth.hex_lattice(n, 0.1, seed=1)), 1)
    code = {"gradient": P.GRADIENT, "divergence": P.DIVERGENCE, "vector": P.DIFFUSION}[kind]
    A = P.Operator(S, code, S.qdata(code), constrained=False,
                   **({"vector": True} if kind == "vector" else {}))
    N = [c * S.ndofs for c in ((1, 3) if kind == "gradient" else (3, 1) if kind == "divergence" else (3, 3))]
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn(N[0], dtype=torch.float64, device="cuda", generator=g)
    want = A.apply(x)
    bufs = [torch.full((k + 9,), float("nan"), dtype=torch.float64, device="cuda") for k in N]
    xs, ys = bufs[0][shift[0]:shift[0] + N[0]], bufs[1][shift[1]:shift[1] + N[1]]
    xs.copy_(x)
    A.apply(xs, ys)
    # the same products, summed per dof over at most 8 elements in another order; on few elements
    # the sums cancel, so against the size of the input's image
    assert float((ys - want).norm()) <= 1e-13 * max(float(want.norm()), float(x.norm()))
    rest = torch.cat([bufs[1][:shift[1]], bufs[1][shift[1] + N[1]:]])
    assert bool(rest.isnan().all())
