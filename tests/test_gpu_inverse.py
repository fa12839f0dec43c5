"""The inverse transform's launches of large grids, and tensors at any float's
address (runs on an MI355X): the store kernel of 128-row workgroups over two,
four and eight 64-column tiles (rows past the last workgroup, a last column
unit of fewer tiles and one of a few columns) and the grids beside its rule,
and the unaligned store and projections in partials.

The reference is the inverse in float64 on the device.  Bar: 1e-6 of its norm.
The float32 products keep W itself exactly, and the correction's two sums of at
most 2048 and 256 terms are off by about 2^-24 sqrt(terms / 4) of their own
size each: below 1e-6 for the correction, and it is smaller than W.
"""

import pytest
import torch

pytestmark = pytest.mark.gpu

gift = pytest.importorskip("paper_2607_07494_amd.gift")
DEV = "cuda"
IN, BOTH = gift.SIDE_INPUT, gift.SIDE_BOTH


@pytest.fixture(scope="module")
def ctx():
    c = gift.Context()
    yield c
    c.close()


def factor(ctx, gen, m, n, r, sides):
    """A factor of random orthonormal bases, and {side: (U, c')} in float64."""
    f = gift.Factor(ctx, m, n, r, sides)
    parts = {}
    for side, dim in ((gift.SIDE_INPUT, n), (gift.SIDE_OUTPUT, m)):
        if sides & side:
            U = torch.linalg.qr(torch.randn((dim, r), generator=gen, dtype=torch.float64))[0].float().to(DEV)
            ci = torch.linspace(0.9, 0.2, r, device=DEV)
            f.import_(side, U.contiguous(), -ci / (1 + ci), ci, torch.ones(1, device=DEV))
            parts[side] = (U.double(), ci.double())
    return f, parts


def inverse(W, parts):
    W = W.double()
    if gift.SIDE_OUTPUT in parts:
        U, c = parts[gift.SIDE_OUTPUT]
        W = W + (U * c) @ (U.T @ W)
    if gift.SIDE_INPUT in parts:
        U, c = parts[gift.SIDE_INPUT]
        W = W + ((W @ U) * c) @ U.T
    return W


def close(out, W, parts):
    want = inverse(W, parts)
    assert torch.isfinite(out).all()
    assert ((out.double() - want).norm() / want.norm()).item() <= 1e-6


def units_of(count, m, n, r):
    """store_units of csrc/k_update.hip: tiles per workgroup of the store
    kernel, 0 where the launch stays on update_kernel."""
    rows, tiles = -(-m // 128) * count, -(-n // 64)
    units = 8
    while units > 2 and rows * -(-tiles // units) < 1024:
        units //= 2
    wgs = rows * -(-tiles // units)
    rounds = -(-wgs // 512)
    idle = rounds * 512 * units / (rows * tiles)
    if r == 64:
        most = 1.05 if units == 2 else 1.44
    else:
        most = 1.4 if rounds < 3 else 1.46 if units == 2 else 1.6
    return units if wgs >= 512 and idle <= most else 0


@pytest.mark.parametrize("count,m,n,r,units", [
    (8, 1061, 1500, 128, 2), (9, 2037, 836, 64, 2),       # 24 and 14 tiles, the last of 28 and 4 columns
    (3, 5465, 2820, 64, 4), (2, 5465, 2820, 128, 4),      # 45 and 25 tiles: a last unit of one
    (5, 6100, 1540, 128, 4),
    (3, 8100, 2820, 64, 8), (8, 8100, 1028, 128, 8),      # last units of five tiles and of one
    (8, 8177, 260, 128, 0), (8, 1061, 1500, 64, 0),       # much of the last round empty
    (4, 1061, 1500, 64, 0),                               # too small
])
def test_store_units(ctx, count, m, n, r, units):
    print(f"[case] inverse count={count} m={m} n={n} r={r} units={units}", flush=True)
    assert units_of(count, m, n, r) == units
    gen = torch.Generator().manual_seed(m + n + r)
    made = [factor(ctx, gen, m, n, r, IN) for _ in range(count)]
    means = [torch.randn((m, n), generator=gen).to(DEV) for _ in range(count)]
    outs = [torch.full((m, n), float("nan"), device=DEV) for _ in range(count)]
    gift.decode_batch(ctx, [f for f, _ in made], means, outs)
    one = torch.full((m, n), float("nan"), device=DEV)
    for i, (f, parts) in enumerate(made):
        close(outs[i], means[i], parts)
        gift.decode(ctx, f, means[i], one)   # its own grid: another kernel, the same sums
        assert torch.equal(one, outs[i])
        f.close()


@pytest.mark.parametrize("m,n,r,sides,at_mean,at_out", [
    (300, 1003, 48, IN, 1, 0), (300, 1003, 16, IN, 0, 3), (77, 515, 128, IN, 2, 1), (1, 7, 1, IN, 1, 1),
    (300, 1024, 64, IN, 1, 0), (300, 1024, 64, IN, 0, 1), (96, 2048, 96, IN, 3, 3),
    (150, 514, 96, BOTH, 1, 2), (203, 333, 32, BOTH, 1, 1), (200, 512, 128, BOTH, 3, 1), (130, 260, 96, BOTH, 0, 1),
])
def test_unaligned_decode(ctx, m, n, r, sides, at_mean, at_out):
    print(f"[case] unaligned decode m={m} n={n} r={r} sides={sides} +{at_mean} +{at_out}", flush=True)
    gen = torch.Generator().manual_seed(m + n + r)
    f, parts = factor(ctx, gen, m, n, r, sides)
    W = torch.empty(m * n + 8, device=DEV)[at_mean:at_mean + m * n].view(m, n)
    W.copy_(torch.randn((m, n), generator=gen))
    flat = torch.full((m * n + 8,), 7.0, device=DEV)
    out = flat[at_out:at_out + m * n].view(m, n)
    gift.decode(ctx, f, W, out)
    close(out, W, parts)
    assert torch.all(flat[:at_out] == 7) and torch.all(flat[at_out + m * n:] == 7)   # nothing beside it
    f.close()


@pytest.mark.parametrize("m,n", [(300, 512), (203, 333), (1500, 260)])
def test_two_sided_store_at_rank_96(ctx, m, n):
    print(f"[case] two-sided store m={m} n={n}", flush=True)
    gen = torch.Generator().manual_seed(m + n)
    f, parts = factor(ctx, gen, m, n, 96, BOTH)
    W = torch.randn((m, n), generator=gen).to(DEV)
    out = torch.full((m, n), float("nan"), device=DEV)
    gift.decode(ctx, f, W, out)
    close(out, W, parts)
    f.close()
