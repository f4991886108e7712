"""The single-launch fit of small dense tensors against the general kernels: sizes where its lane groups, column pieces and
arrays have remainders, many slices of few entities (columns one at a time: padded to four they exceed the LDS), ranks up to
the number of entities.  Both sum in fp32 in a different order: a few 2^-24 per sum and iteration; ten iterations leave 2^-17 as a bar."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,m,k,q", [(1, 1, 1, 2), (2, 3, 2, 3), (5, 1, 4, 1), (17, 2, 5, 9), (63, 3, 3, 2), (64, 8, 1, 2),
                                     (20, 80, 1, 2), (64, 1, 56, 1), (33, 4, 16, 3), (30, 5, 30, 2),
                                     # rows spaced in LDS (16, 32), not spaced for want of room, one column at a time
                                     (16, 2, 16, 2), (40, 4, 32, 2), (34, 5, 30, 2), (64, 7, 7, 2), (31, 15, 13, 2), (62, 8, 5, 2)])
@pytest.mark.parametrize("delta", [0.0, 0.03])
def test_single_launch_fit_against_general_kernels(lib, n, m, k, q, delta):
    g = torch.Generator(device=DEV)
    g.manual_seed(n * 7 + k)
    X = torch.rand((m, n, n), generator=g, device=DEV) + 0.1
    got = []
    for fused in (True, False):
        h = lib.nnrescal_init(lib.DenseX(X), k=k, q=q, delta=delta, seed=4, fused_small=fused)
        lib.nnrescal_fit(h, 10)
        got.append([f.double() for f in lib.nnrescal_get_factors(h)])
        lib.nnrescal_destroy(h)
    for a, b in zip(*got):
        for r in range(q):
            assert ((a[r] - b[r]).norm() / b[r].norm()).item() <= 2.0 ** -17, (n, m, k, q, delta, r)
