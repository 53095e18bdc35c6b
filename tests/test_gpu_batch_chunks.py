"""Batched applies: one workgroup per tile and chunk of right-hand sides, over meshes of
several orders and sizes, against the single applies."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [2, 4, 6, 8, 16, 24, 514])
@pytest.mark.parametrize("kind", ["mass", "diffusion"])
@pytest.mark.parametrize("f32", [False, True])
def test_every_tile_on_uneven_meshes(nrhs, kind, f32):
    import torch
    from paper_1911_09220_amd import pafem as P
    code = P.MASS if kind == "mass" else P.DIFFUSION
    ops, xs = [], []
    g = torch.Generator(device="cuda").manual_seed(1)
    sizes = [(1, (1, 1, 1)), (1, (3, 2, 2)), (2, (3, 1, 2)), (3, (2, 2, 1)), (4, (2, 1, 1)), (5, (1, 2, 1)), (6, (2, 1, 1))]
    for k, (p, n) in enumerate(sizes):
        S = P.Space(P.Mesh.from_dict(synth.hex_lattice(n, 0.1, seed=k, rotate_seed=k)), p, renumber=bool(k % 2))
        qd = S.qdata(code)
        dt = torch.float32 if f32 else torch.float64
        if f32:
            qd = P.lowered_qdata(qd, P.F32)
        ops.append(P.Operator(S, code, qd, constrained=bool(k % 3), qdata_dtype=P.F32 if f32 else P.F64))
        xs.append(torch.randn(S.ndofs, nrhs, dtype=dt, device="cuda", generator=g))
    B = P.Batch(ops, nrhs)
    want = [torch.stack([o.apply(x[:, j].contiguous()) for j in range(nrhs)], dim=1) for o, x in zip(ops, xs)]
    tiles = {}
    for p in {p for p, _ in sizes}:
        for c in range(6):
            try:
                B.set_tile(p, c)
                tiles.setdefault(p, []).append(c)
            except P.PafemError:
                pass
        B.set_tile(p, -1)
    assert all(4 in t for t in tiles.values())
    for r in range(max(len(t) for t in tiles.values())):
        for p, t in tiles.items():
            B.set_tile(p, t[r % len(t)])
        ys = [torch.full_like(x, float("nan")) for x in xs]
        B.apply(xs, ys)
        for y, w in zip(ys, want):
            # sums of at most 8 elements' (p+1)^3 terms in another order
            tol = 2e-5 if f32 else 1e-13
            assert float((y - w).norm()) <= tol * float(w.norm())
