"""Batched applies whose workgroups walk several chunks of right-hand sides (small tiles at
p <= 3): all chunks, groups of them of even and uneven size, and one each, against single applies."""
import pytest

import synth

pytestmark = pytest.mark.gpu


# 4096 tiles and more: all chunks in one workgroup; 2197: two groups; 1000: five; 36: one each
@pytest.mark.parametrize("n", [(16, 16, 16), (13, 13, 13), (10, 10, 10), (3, 3, 4)])
@pytest.mark.parametrize("nrhs,tile", [(6, 4), (10, 4), (54, 4), (20, 0), (36, 0)])
@pytest.mark.parametrize("p", [1, 2, 3])
@pytest.mark.parametrize("kind,f32", [("diffusion", False), ("diffusion", True), ("mass", False)])
def test_walking_workgroups(n, nrhs, tile, p, kind, f32):
    import torch
    from paper_1911_09220_amd import pafem as P
    code = P.MASS if kind == "mass" else P.DIFFUSION
    dt = torch.float32 if f32 else torch.float64
    g = torch.Generator(device="cuda").manual_seed(1)
    ops, xs = [], []
    for k, size in enumerate((n, (2, 1, 2))):
        S = P.Space(P.Mesh.from_dict(synth.hex_lattice(size, 0.1, seed=k, rotate_seed=k)), p)
        qd = S.qdata(code)
        if f32:
            qd = P.lowered_qdata(qd, P.F32)
        ops.append(P.Operator(S, code, qd, constrained=k == 0, qdata_dtype=P.F32 if f32 else P.F64))
        xs.append(torch.randn(S.ndofs, nrhs, dtype=dt, device="cuda", generator=g))
    B = P.Batch(ops, nrhs)
    B.set_tile(p, tile)
    ys = [torch.full_like(x, float("nan")) for x in xs]
    B.apply(xs, ys)
    for o, x, y in zip(ops, xs, ys):
        for j in range(nrhs):
            w = o.apply(x[:, j].contiguous())
            # sums of at most 8 elements' (p+1)^3 terms in another order
            assert float((y[:, j] - w).norm()) <= (2e-5 if f32 else 1e-13) * float(w.norm())
