"""The k x k steps of the factor refresh (runs on an MI355X): the register-tile
Cholesky and inverse up to 256 and the block Jacobi eigensolver for
64 < k <= 256, at the edges of their 16-wide tiles, 32-wide column blocks and
kernel ranges.

Both are float64 inside.  The Cholesky factors are compared with numpy's of the
same float32 statistics (exported through a Cholesky-form factor): R is stored
in float32, so a relative error of 2^-23 per entry plus the statistics' own
rounding over the input's condition number (about 1e3), 1e-3 as the other
Cholesky tests take.  The eigensolver is compared through S^-1's action with
the float64 mirror of the refresh (1e-3, the refresh tests' bound).
"""

import numpy as np
import pytest
import torch

from oracle import codec, subspace
from synth import factor_inputs, haar
from test_gpu_factor import action_gap, ctx, exported, say, t  # noqa: F401

pytestmark = pytest.mark.gpu

gift = pytest.importorskip("paper_2607_07494_amd.gift")


@pytest.mark.parametrize("dim,block", [(1, 0), (15, 0), (16, 0), (17, 0), (33, 0), (127, 0), (128, 0), (129, 0),
                                       (144, 0), (241, 0), (256, 0), (257, 0), (300, 150), (70, 17)])
def test_cholesky_tiles(ctx, dim, block):  # noqa: F811
    say(f"chol tiles dim={dim} block={block}")
    x = factor_inputs(400 + dim, 4 * dim, dim)[0]
    ref = codec.chol_factor(codec.factor_statistics(x), block, 1e-4)
    f = gift.CholFactor(ctx, 4, dim, block, gift.SIDE_INPUT, 1e-4)
    f.update(acts=t(x))
    R, Ri = (v.cpu().numpy().astype(np.float64) for v in f.export(gift.SIDE_INPUT))
    for got, want in ((R, ref.R), (Ri, ref.Rinv)):
        assert np.linalg.norm(got - want) <= 1e-3 * np.linalg.norm(want)
        assert np.all(np.tril(got, -1) == 0)
    f.close()


@pytest.mark.parametrize("dim,r", [(100, 33), (128, 64), (129, 64), (320, 65), (150, 100), (320, 97), (250, 125),
                                   (512, 128), (400, 129)])
def test_eigensolver_blocks(ctx, dim, r):  # noqa: F811
    """Cold, then warm on other tokens (k = min(dim, 2 r) from 66 to 258)."""
    say(f"block eigensolver dim={dim} r={r}")
    X, _ = factor_inputs(500 + dim, 4 * dim, dim)
    X2, _ = factor_inputs(500 + dim, 3 * dim, dim)
    f = gift.Factor(ctx, 16, dim, r, gift.SIDE_INPUT, seed=dim)
    f.update(acts=t(X), iters=3)
    A = codec.factor_statistics(X)
    mirror, _ = subspace.subspace_factor(A, r, 3, seed=dim)
    got = exported(f, gift.SIDE_INPUT)
    assert action_gap(got, mirror, dim) <= 1e-3
    np.testing.assert_allclose(got.U.T @ got.U, np.eye(r), atol=1e-5)
    f.update(acts=t(X2), iters=2)
    got = exported(f, gift.SIDE_INPUT)
    np.testing.assert_allclose(got.U.T @ got.U, np.eye(r), atol=1e-5)
    A2 = codec.factor_statistics(X2)
    w = np.sort(np.linalg.eigvalsh(A2))[::-1]
    assert np.trace(got.U.T @ A2 @ got.U) / w[:r].sum() >= 0.999
    f.close()


def test_eigensolver_degenerate_spectra(ctx):  # noqa: F811
    """A spectrum of two values (every gap zero or large), fewer tokens than the
    dimension, and no statistics at all."""
    dim, r = 160, 33
    rng = np.random.default_rng(3)
    spec = np.where(np.arange(dim) < r, 4.0, 1.0)
    X = ((haar(rng, 4 * dim, dim) * np.sqrt(4 * dim)) * np.sqrt(spec) @ haar(rng, dim, dim).T).astype(np.float32)
    f = gift.Factor(ctx, 16, dim, r, gift.SIDE_INPUT, seed=5)
    f.update(acts=t(X), iters=12)
    got, exact = exported(f, gift.SIDE_INPUT), codec.lowrank_factor(codec.factor_statistics(X), r)
    assert action_gap(got, exact, dim) <= 1e-3
    assert got.sigma2 == pytest.approx(1.0, rel=1e-4)
    f.close()
    Y = rng.standard_normal((80, dim)).astype(np.float32)
    f = gift.Factor(ctx, 16, dim, r, gift.SIDE_INPUT, damping=1e-3, seed=6)
    f.update(acts=t(Y), iters=2)
    got = exported(f, gift.SIDE_INPUT)
    mirror, _ = subspace.subspace_factor(codec.factor_statistics(Y), r, 2, seed=6, damping=1e-3)
    assert action_gap(got, mirror, dim) <= 1e-3
    # all-zero statistics: the identity
    f.update(acts=torch.zeros((80, dim), device="cuda"), iters=1)
    got = exported(f, gift.SIDE_INPUT)
    assert np.all(got.c_fwd == 0) and np.all(got.c_inv == 0) and got.sigma2 == 0.0
    f.close()


def same_factor(a, b):
    for x, y in zip(a.export(gift.SIDE_INPUT), b.export(gift.SIDE_INPUT)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("dim,r,iters", [(96, 16, 2), (96, 16, 0), (160, 33, 2), (320, 80, 1), (300, 129, 1)])
@pytest.mark.parametrize("bad", [0.0, float("nan")])
def test_statistics_without_a_trace(ctx, dim, r, iters, bad):  # noqa: F811
    """A refresh on all-zero (or not finite) statistics, first and after
    another one, for every solver range: the identity in every layout, and the
    next refresh goes on from the basis there was (k = 32, 66, 160, 258)."""
    say(f"no trace dim={dim} r={r} iters={iters} bad={bad}")
    X, _ = factor_inputs(700 + dim, 2 * dim, dim)
    X2, _ = factor_inputs(701 + dim, 2 * dim, dim)
    none = torch.full((2 * dim, dim), bad, device="cuda")
    m, N = 24, 2
    g = torch.randn((N, m, dim), device="cuda")

    def codes_of(f):
        codes = torch.empty((N, m, dim), dtype=torch.uint8, device="cuda")
        scales = torch.empty((N, 1, 1), device="cuda")
        gift.encode(ctx, f, g, codes, scales)
        mean, out = torch.empty((m, dim), device="cuda"), torch.empty((m, dim), device="cuda")
        gift.reduce_local(ctx, codes, scales, mean)
        gift.decode(ctx, f, mean, out)
        return codes, scales, mean, out

    def check_identity(f):
        U, cf, ci, s2 = f.export(gift.SIDE_INPUT)
        for v in (U, cf, ci, s2):
            assert torch.all(v == 0)
        got, want = codes_of(f), codes_of(None)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        assert torch.equal(got[3], got[2])

    f, fresh = (gift.Factor(ctx, m, dim, r, gift.SIDE_INPUT, seed=dim) for _ in range(2))
    f.update(acts=none, iters=iters)
    check_identity(f)
    # beside a member with statistics, in one call
    gift.factor_update_batch(ctx, [f, fresh], [none, t(X)], [None, None], iters=iters)
    check_identity(f)
    f.update(acts=t(X), iters=iters)
    same_factor(f, fresh)
    f.update(acts=none, iters=iters)
    check_identity(f)
    for x in (f, fresh):
        x.update(acts=t(X2), iters=iters)
    same_factor(f, fresh)
    f.close()
    fresh.close()


@pytest.mark.parametrize("dim,r", [(4096, 128), (4096, 72), (4092, 80), (2052, 112), (4096, 120), (4096, 48)])
def test_product_chains(ctx, dim, r):  # noqa: F811
    """Q A at k > 128 sums its contraction in four chains, not one.  1024 tokens
    of 1, 2 and 3 give exact statistics, all positive, with one dominant
    eigenvector, each entry of which then carries the rounding of its own sum
    of `dim` terms of one sign.  n roundings of a partial sum that grows evenly
    to S leave S u sqrt(n / 3) / sqrt(3) (u = 2^-24, a rounding's error
    uniform); the matrix core rounds once per product, or less often.  Measured:
    one chain 8.3e-7 at 4092, four 2.2e-7, the bound 0.6 of one chain's
    estimate at a rounding per four products.  (k = 96 runs split-bf16
    products: 2^-16 each, of random sign.)"""
    say(f"product chains dim={dim} r={r}")
    rng = np.random.default_rng(dim + r)
    X = rng.integers(1, 4, (1024, dim)).astype(np.float64)
    f = gift.Factor(ctx, 16, dim, r, gift.SIDE_INPUT, seed=1)
    f.update(acts=t(X.astype(np.float32)), iters=3)
    u = exported(f, gift.SIDE_INPUT).U[:, 0]
    v = np.ones(dim)
    for _ in range(40):
        v = X.T @ (X @ v)
        v /= np.linalg.norm(v)
    err = np.linalg.norm(u * np.sign(u.sum()) / np.linalg.norm(u) - v)
    one = 2.0 ** -24 * np.sqrt(dim / 4 / 3) / np.sqrt(3)
    say(f"  error {err:.3g}, one chain {one:.3g}")
    assert err <= (0.6 * one if r > 64 else 2.0 ** -16 / np.sqrt(3 * dim) * 4 + one)
    f.close()


@pytest.mark.parametrize("dim,r,count,chains", [(4092, 128, 4, 4), (4092, 96, 4, 4), (4096, 128, 16, 1)])
def test_product_of_several_factors(ctx, dim, r, count, chains):  # noqa: F811
    """Q A at k > 128 in workgroups of two strips per wave: each factor's
    leading eigenvector as in test_product_chains (the statistics of factor i
    are those of factor 0 with its features moved i places), and a batch of
    4096 16-row strips, whose sums are one chain (its own estimate for a
    rounding per product)."""
    say(f"product of {count} factors dim={dim} r={r}")
    rng = np.random.default_rng(dim + r)
    X = rng.integers(1, 4, (1024, dim)).astype(np.float64)
    v = np.ones(dim)
    for _ in range(40):
        v = X.T @ (X @ v)
        v /= np.linalg.norm(v)
    fs = [gift.Factor(ctx, 16, dim, r, gift.SIDE_INPUT, seed=1 + i) for i in range(count)]
    x = t(X.astype(np.float32))
    gift.factor_update_batch(ctx, fs, [torch.roll(x, 37 * i, 1).contiguous() for i in range(count)],
                             [None] * count, iters=3)
    one = 2.0 ** -24 * np.sqrt(dim / 4 / 3) / np.sqrt(3)
    for i, f in enumerate(fs):
        u = exported(f, gift.SIDE_INPUT).U[:, 0]
        err = np.linalg.norm(u * np.sign(u.sum()) / np.linalg.norm(u) - np.roll(v, 37 * i))
        say(f"  factor {i}: error {err:.3g}, one chain {one:.3g}")
        assert err <= (0.6 * one if chains == 4 else 2 * one)
        f.close()
