"""A batched apply of more threads than one launch may have (2^32): 1e6 elements at p = 1 with
480 right-hand sides, against the same columns 16 at a time."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [0, 2])
def test_more_threads_than_a_launch(tile):
    import torch
    from paper_1911_09220_amd import pafem as P
    n, nrhs = 100, 480
    assert n ** 3 * 9 * nrhs > 2 ** 32
    S = P.Space(P.Mesh.from_dict(synth.hex_lattice(n, 0.05, seed=1)), 1)
    A = P.Operator(S, P.DIFFUSION, S.qdata(P.DIFFUSION))
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(S.ndofs, 16, dtype=torch.float64, device="cuda", generator=g)
    want = torch.empty_like(x)
    P.Batch([A], 16).apply([x], [want])
    xs = x.repeat(1, nrhs // 16)
    xs[:, 464:] *= 2.0  # the last columns are others
    ys = torch.full_like(xs, float("nan"))
    B = P.Batch([A], nrhs)
    B.set_tile(1, tile)
    B.apply([xs], [ys])
    for c in range(0, nrhs, 16):
        y = ys[:, c:c + 16] / (2.0 if c >= 464 else 1.0)
        # sums of at most 8 elements' 8 terms in another order
        assert float((y - want).norm()) <= 1e-13 * float(want.norm())
