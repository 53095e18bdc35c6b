"""The solvers' vector kernels at the sizes where their grids and partial sums change: less
than one workgroup, several, all, and more element energies than every workgroup sums itself."""
import pytest

import synth

pytestmark = pytest.mark.gpu


# p = 1, 100^3: 35715 apply tiles, so the energies are folded first
@pytest.mark.parametrize("p,n", [(1, 2), (2, 5), (1, 10), (3, 8), (2, 40), (1, 100)])
@pytest.mark.parametrize("scatter", ["atomic", "evec"])
@pytest.mark.parametrize("constrained", [True, False])
def test_pcg_iterates_equal_plain_cg(p, n, scatter, constrained):
    import torch
    from paper_1911_09220_amd import pafem as P
    S = P.Space(P.Mesh.from_dict(synth.hex_lattice(n, 0.05, seed=1)), p)
    kind = P.DIFFUSION if constrained else P.MASS
    A = P.Operator(S, kind, S.qdata(kind), constrained=constrained, scatter=scatter)
    g = torch.Generator(device="cuda").manual_seed(3)
    b = torch.randn(S.ndofs, dtype=torch.float64, device="cuda", generator=g)
    diag = A.diagonal()
    x = torch.randn(S.ndofs, dtype=torch.float64, device="cuda", generator=g)
    ref = x.clone()
    got, info = A.pcg(b, x=x, diag=diag, rel_tol=0.0, max_iter=5, check_every=2)
    r = b - A.apply(ref)
    z = r / diag
    d, rz, hist = z.clone(), r @ z, [float(r.norm() / b.norm())]
    for _ in range(5):
        if float(rz) == 0.0:
            break
        q = A.apply(d)
        alpha = rz / (d @ q)
        ref += alpha * d
        r -= alpha * q
        z = r / diag
        rz, old = r @ z, rz
        d = z + (rz / old) * d
        hist.append(float(r.norm() / b.norm()))
    # one free dof (1, 2): the first step is exact and may leave no residual at all
    assert (info["iters"] == 5 and info["status"] == "ENOTCONV") or info["rel_res"] == 0.0
    # five iterations of FP64 sums of at most 1e6 terms: 5 * 1e6 * 2^-53 < 1e-9 at the very worst
    assert float((got - ref).norm() / ref.norm()) < 1e-9
    # the history is relative to ||b|| already (after an exact solve it is rounding alone)
    assert max(abs(a - c) for a, c in zip(info["history"], hist)) < 1e-9
