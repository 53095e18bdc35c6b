"""Which solver batches are captured (8 to 64 kernels, 16 replays allowed): counts on both sides of
each limit, and the captured solves against direct launches."""
import pytest

import synth

pytestmark = pytest.mark.gpu


def _replays(fn):
    from paper_1911_09220_amd import pafem as P
    before = P.pafem_graph_replays()
    out = fn()
    return P.pafem_graph_replays() - before, out


def _both(fn):
    """Replays and result under graph mode, and the result of direct launches."""
    from paper_1911_09220_amd import pafem as P
    prev = P.pafem_set_graph_mode(1)
    try:
        n, out = _replays(fn)
        P.pafem_set_graph_mode(0)
        none, direct = _replays(fn)
    finally:
        P.pafem_set_graph_mode(prev)
    assert none == 0
    return n, out, direct


def _same(out, direct):
    (x, i), (xd, d) = out, direct
    assert i["status"] == d["status"] and abs(i["iters"] - d["iters"]) <= 1
    # the atomic sums of an apply are unordered
    assert float((x - xd).norm()) <= 1e-10 * float(xd.norm())


# kernels a batch: direction in the apply 2 check + 1, element vectors 4 check
@pytest.mark.parametrize("scatter,check,max_iter,captured",
                         [("atomic", 3, 300, False), ("atomic", 4, 300, True), ("atomic", 31, 600, True),
                          ("atomic", 32, 600, False), ("atomic", 4, 63, False), ("atomic", 4, 64, True),
                          ("evec", 1, 300, False), ("evec", 2, 300, True), ("evec", 16, 300, True),
                          ("evec", 17, 300, False)])
def test_pcg_batches(scatter, check, max_iter, captured):
    from paper_1911_09220_amd import pafem as P
    S = P.Space(P.Mesh.from_dict(synth.hex_lattice(6, 0.1, seed=3)), 2)
    A = P.Operator(S, P.DIFFUSION, S.qdata(P.DIFFUSION), scatter=scatter)
    b, diag = S.linear_form(P.SOURCE_SINE), A.diagonal()
    n, out, direct = _both(lambda: A.pcg(b, diag=diag, rel_tol=1e-10, max_iter=max_iter, check_every=check))
    assert (n > 0) == captured
    _same(out, direct)


# two levels, degree 1: an iteration is 15 kernels and 2 for each of the coarse solve
@pytest.mark.parametrize("coarse,max_iter,captured", [(1, 200, True), (8, 200, True), (9, 200, False), (4, 31, False), (4, 32, True)])
@pytest.mark.parametrize("check", [2, 5])
def test_multigrid_pairs(coarse, max_iter, captured, check):
    import torch
    from paper_1911_09220_amd import pafem as P
    M = P.Mesh.from_dict(synth.hex_lattice(6, 0.1, seed=5))
    ops, diags, lmax = [], [], []
    for q in (2, 1):
        S = P.Space(M, q)
        op = P.Operator(S, P.DIFFUSION, S.qdata(P.DIFFUSION))
        d = op.diagonal()
        v = torch.as_tensor(synth.hash_normal(S.dof_coords(), seed=q), device="cuda")
        ops.append(op)
        diags.append(d)
        lmax.append(op.lambda_max(d, v, 20))
    G = P.PMG(ops, diags, lmax, degree=1, coarse_iters=coarse)
    b = ops[0].space.linear_form(P.SOURCE_SINE)
    n, out, direct = _both(lambda: G.fcg(b, rel_tol=1e-10, max_iter=max_iter, check_every=check))
    assert (n > 0) == captured
    _same(out, direct)
