"""The dense pass over X keeps its fp32 operands as sums of three bf16 terms.  Both products of a slice against 64-bit
products of the explicitly perturbed tensor (`nnrescal_perturb`, which the parity tests hold to the oracle bit for bit),
member by member and column by column, at the edges of its tiles and panels (narrow and wide), for delta = 0, small and
large, with factors of both signs and columns and tensors of very different size.

Bar per member and column of sums, relative to the column's norm: single products are within 2^-21.4 (below), random in
sign; the fp32 sums of n terms add about sqrt(n) 2^-24.  That bar grows with n while the errors of the terms average out,
so a lost low-order term is looked for where every result is ONE product: X with one entry per row and column.

Bar per product: its operands are held exactly; the two term products that are left out are below 2^-23 each, and three
accumulating instructions and a final sum may cut a unit of 2^-24 each: 1.5 * 2^-22.  The root mean square over thousands
of products is 2^-24.8 by measurement (2^-25.2 is the rounding of the result alone); with 2^-24.5 as a bar, an operand
held to 2^-22 instead of 2^-24 fails, and so does any lost term (2^-17 or more)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(lib, n, m, k, q, delta, deterministic=False, xscale=1.0, signs=False):
    g = torch.Generator(device=DEV)
    g.manual_seed(n * 131 + k)
    X = torch.rand((m, n, n), generator=g, device=DEV) * xscale
    A = torch.rand((q, n, k), generator=g, device=DEV) + 0.01
    if signs:
        A = A - 0.5
    A = A * (2.0 ** torch.linspace(-30, 30, k, device=DEV))            # columns of very different size
    R = torch.ones((q, m, k, k), device=DEV)
    h = lib.nnrescal_init(lib.DenseX(X), k=k, q=q, delta=delta, seed=n, A0=A.contiguous(), R0=R, deterministic=deterministic)
    tol = 2.0 ** -20 + n ** 0.5 * 2.0 ** -23
    for t in range(m):
        P, Q = lib.nnrescal_products(h, t)
        for r in range(q):
            Xr = lib.nnrescal_perturb(lib.DenseX(X), r, delta, n)[t].double() if delta > 0 else X[t].double()
            a = A[r].double()
            size = (Xr.abs() @ a.abs()).norm(dim=0), (Xr.abs().T @ a.abs()).norm(dim=0)
            for got, want, scale in ((P[r], Xr @ a, size[0]), (Q[r], Xr.T @ a, size[1])):
                err = ((got.double() - want).norm(dim=0) / scale).max().item()
                assert err <= tol, (n, m, k, q, delta, t, r, err, tol)
    lib.nnrescal_destroy(h)


@pytest.mark.parametrize("n,m,k,q", [(1, 1, 1, 3), (1, 5, 1, 9), (2, 1, 2, 4), (3, 2, 3, 5), (15, 2, 4, 8), (17, 1, 16, 6),
                                     (127, 2, 16, 11), (129, 1, 17, 7), (255, 1, 33, 3), (258, 2, 64, 2), (385, 1, 32, 3)])
@pytest.mark.parametrize("delta", [0.0, 0.0625, 0.07, 0.9])
def test_products_at_tile_edges(lib, n, m, k, q, delta):
    _check(lib, n, m, k, q, delta)


@pytest.mark.parametrize("n,k,q,delta,det", [(4097, 16, 7, 0.03, False), (4225, 5, 2, 0.5, False), (4099, 40, 1, 0.03, True),
                                             (4096, 12, 1, 0.0, True)])
def test_products_with_wide_panels(lib, n, k, q, delta, det):
    _check(lib, n, 1, k, q, delta, deterministic=det)


@pytest.mark.parametrize("xscale", [1e-30, 1e25])
def test_products_range_and_signs(lib, xscale):
    _check(lib, 200, 1, 16, 5, 0.03, xscale=xscale)
    _check(lib, 200, 1, 20, 3, 0.03, xscale=xscale, signs=True)


# larger ensembles, several slices (a call of nnrescal_products is a launch for ONE slice)
@pytest.mark.parametrize("n,m,k,q", [(100, 2, 8, 4), (250, 3, 10, 9), (333, 5, 8, 9), (333, 5, 24, 9), (500, 8, 3, 15),
                                     (600, 4, 24, 9), (600, 4, 40, 5), (600, 7, 16, 16), (1501, 8, 3, 9)])
@pytest.mark.parametrize("delta", [0.0, 0.03, 0.5])
def test_products_in_every_form(lib, n, m, k, q, delta):
    _check(lib, n, m, k, q, delta)


def _check_single_products(lib, n, k, q, delta, deterministic=False, signs=False):
    g = torch.Generator(device=DEV)
    g.manual_seed(n + 7 * k + q)
    X = torch.zeros((1, n, n), device=DEV)
    rows, pi = torch.arange(n, device=DEV), torch.randperm(n, generator=g, device=DEV)
    X[0, rows, pi] = 1.0 + torch.rand(n, generator=g, device=DEV)
    A = 1.0 + torch.rand((q, n, k), generator=g, device=DEV)
    if signs:
        A = A * torch.where(torch.rand((q, n, k), generator=g, device=DEV) < 0.5, -1.0, 1.0)
    R = torch.ones((q, 1, k, k), device=DEV)
    h = lib.nnrescal_init(lib.DenseX(X), k=k, q=q, delta=delta, seed=n, A0=A, R0=R, deterministic=deterministic)
    P, Q = lib.nnrescal_products(h, 0)
    lib.nnrescal_destroy(h)
    errs = []
    for r in range(q):
        x = (lib.nnrescal_perturb(lib.DenseX(X), r, delta, n)[0] if delta > 0 else X[0])[rows, pi].double()[:, None]
        a = A[r].double()
        want_p, want_q = x * a[pi], torch.empty_like(a)
        want_q[pi] = x * a
        errs.append(torch.stack([((P[r].double() - want_p) / want_p).abs(), ((Q[r].double() - want_q) / want_q).abs()]))
    err = torch.stack(errs)
    for which in (0, 1):
        worst, rms = err[:, which].max().item(), err[:, which].square().mean().sqrt().item()
        assert worst <= 1.5 * 2.0 ** -22 and (rms <= 2.0 ** -24.5 or n * q * k < 1000), (n, k, q, delta, "PQ"[which], worst, rms)


# (n, k, q) of one slice: every kernel that the plan of a pass can choose (test_dense_plan.py holds the list to that)
FORMS = [(17, 3, 1), (333, 8, 10), (700, 16, 8), (2001, 16, 1), (2001, 16, 2), (1000, 16, 15), (2176, 16, 8), (4200, 16, 13), (6001, 16, 9),
         (6000, 16, 10), (6001, 16, 11), (33, 17, 2), (1001, 24, 2), (1001, 24, 7), (2502, 32, 4), (6001, 24, 5), (6000, 24, 6),
         (300, 40, 5), (2001, 40, 2), (3000, 40, 3), (6001, 40, 5), (640, 64, 3), (2001, 64, 1), (2500, 64, 2), (6001, 64, 3), (2001, 40, 6),
         (3000, 64, 4)]


@pytest.mark.parametrize("n,k,q", FORMS)
@pytest.mark.parametrize("delta", [0.0, 0.03, 0.5])
def test_single_products(lib, n, k, q, delta):
    _check_single_products(lib, n, k, q, delta)


@pytest.mark.parametrize("n,k,q", [(130, 8, 4), (2176, 16, 8)])
@pytest.mark.parametrize("delta", [1e-6, 0.005, 0.0624, 0.0625, 0.07, 0.99])
def test_single_products_for_any_delta(lib, n, k, q, delta):
    _check_single_products(lib, n, k, q, delta)


def test_single_products_signs_and_reproducible(lib):
    _check_single_products(lib, 300, 16, 8, 0.03, signs=True)
    _check_single_products(lib, 300, 16, 8, 0.03, deterministic=True)


@pytest.mark.parametrize("n,m,k,q", [(90, 6, 5, 3), (600, 5, 16, 13), (600, 5, 24, 6), (500, 3, 40, 3), (300, 7, 64, 2), (1500, 4, 16, 8)])
@pytest.mark.parametrize("delta", [0.0, 0.03])
def test_single_products_in_one_launch_for_all_slices(lib, n, m, k, q, delta):
    """An iteration's launch covers all slices.  X_t with one entry per row and column and R_t = 0 but for one slice s, where it is
    diagonal (zeros stay), leave (P_s + Q_s)[i][c], two products, in the new A[i][c] = A R_s (P_s + Q_s) / (A W).  Against one
    iteration in 64 bits, element by element: 2^-21.4 of the products, and a few 2^-23 each of R (a quotient of sums), W and
    the quotient: 2^-20.  A lost term is 2^-17 or more."""
    g = torch.Generator(device=DEV)
    g.manual_seed(n + m)
    rows = torch.arange(n, device=DEV)
    X = torch.zeros((m, n, n), device=DEV)
    for t in range(m):
        X[t, rows, torch.randperm(n, generator=g, device=DEV)] = 1.0 + torch.rand(n, generator=g, device=DEV)
    A = 1.0 + torch.rand((q, n, k), generator=g, device=DEV)
    Xq = [(lib.nnrescal_perturb(lib.DenseX(X), r, delta, 7) if delta > 0 else X) for r in range(q)]
    for s in range(m):
        R = torch.zeros((q, m, k, k), device=DEV)
        R[:, s] = torch.eye(k, device=DEV)
        h = lib.nnrescal_init(lib.DenseX(X), k=k, q=q, delta=delta, seed=7, A0=A, R0=R, fused_small=False)
        lib.nnrescal_mu_step(h)
        got, _ = lib.nnrescal_get_factors(h)
        lib.nnrescal_destroy(h)
        for r in range(q):
            x, a, rt = Xq[r][s].double(), A[r].double(), R[r, s].double()
            gram = a.T @ a
            rt = rt * (a.T @ (x @ a)) / (gram @ rt @ gram)
            num = (x @ a) @ rt.T + (x.T @ a) @ rt
            want = a * num / (a @ (rt @ gram @ rt.T + rt.T @ gram @ rt))
            err = ((got[r].double() - want) / want).abs().max().item()
            assert err <= 2.0 ** -20, (n, m, k, q, delta, s, r, err)
