"""The codec on rows of any length and tensors at any float's address (runs on
an MI355X): the register-direct update kernel with rows that are no multiple of
four (its last lane's columns cross the end of the row), ranks 48 and 96, the
projection in partials, the tile kernel at the other ranks, and the rank sum.

Bars as in the codec tests: codes, scales, residuals, counters and rank mean
bit for bit the oracle's on the stored W~, W~ and the decode within 1e-5 of
float64 (float32 products give about 1e-7 here, held at 1e-6 where the start's
precision could be lost).
"""

import numpy as np
import pytest
import torch

from oracle import codec
from synth import gradient_set
from test_gpu_codec import ctx, gpu_decode, gpu_reduce, make_factor, rel, say, t  # noqa: F401

pytestmark = pytest.mark.gpu

gift = pytest.importorskip("paper_2607_07494_amd.gift")
DEV = "cuda"
IN, OUT, BOTH = gift.SIDE_INPUT, gift.SIDE_OUTPUT, gift.SIDE_BOTH


def placed(x, shift):
    """x on the GPU, `shift` elements past an aligned address."""
    flat = torch.empty(x.size + shift, dtype=torch.from_numpy(x).dtype, device=DEV)
    v = flat[shift:].view(x.shape)
    v.copy_(t(x))
    return v


@pytest.mark.parametrize("N,m,n,r,sides,br,bc,ef,shared,shift", [
    (2, 130, 129, 16, IN, 0, 0, False, False, 0),
    (3, 65, 262, 48, IN, 0, 128, True, False, 0),
    (2, 63, 191, 48, OUT, 0, 64, False, True, 0),
    (2, 128, 643, 96, IN, 64, 100, True, False, 0),
    (2, 200, 333, 32, BOTH, 0, 0, True, False, 0),
    (2, 150, 514, 128, BOTH, 0, 128, False, False, 0),
    (5, 100, 1027, 64, IN, 7, 9, False, False, 0),
    (1, 33, 5, 4, IN, 0, 0, False, False, 0),       # tile kernel, rows shorter than its vectors
    (2, 77, 131, 40, IN, 0, 50, True, True, 0),     # tile kernel (rank 40)
    (2, 96, 1030, 24, IN, 0, 0, False, False, 0),   # partials of the tile kernel
    (2, 96, 512, 64, IN, 0, 128, True, False, 1),   # aligned rows at an odd address
    (2, 96, 512, 48, IN, 0, 128, False, False, 3),
    (2, 64, 96, 0, 0, 0, 32, True, False, 2),       # Euclidean
    (2, 61, 99, 0, 0, 5, 7, False, True, 0),
])
def test_ragged_codec(ctx, N, m, n, r, sides, br, bc, ef, shared, shift):  # noqa: F811
    say(f"ragged codec N={N} m={m} n={n} r={r} sides={sides} block=({br},{bc}) ef={ef} shared={shared} +{shift}")
    grads = gradient_set(900 + m, 901 + n, N, m, n)
    f, fA, fG = make_factor(ctx, m, n, r, sides, seed=m + n) if r else (None, None, None)
    mode = gift.SCALE_SHARED if shared else gift.SCALE_LOCAL
    R0 = (gradient_set(902 + m, 903, N, m, n) * np.float32(0.01)) if ef else None
    g = placed(grads, shift)
    nbr, nbc = gift.scale_grid(m, n, br, bc)
    hits = torch.zeros((N, 2), dtype=torch.int32, device=DEV)
    out = []
    for store in (True, False):
        codes = placed(np.full((N, m, n), 0x55, np.uint8), shift)
        scales = torch.full((N, nbr, nbc), float("nan"), device=DEV)
        R = placed(R0, shift) if ef else None
        tr = placed(np.zeros((N, m, n), np.float32), shift) if store else None
        gift.encode(ctx, f, g, codes, scales, br, bc, mode, ef=R, transformed=tr, hits=hits if store else None)
        torch.cuda.synchronize()
        out.append([None if v is None else v.cpu().numpy() for v in (codes, scales, R, tr)])
    (codes, scales, R, tr), (codes2, scales2, R2, _) = out
    want = codec.forward(grads, fA, fG) if r else grads.astype(np.float64)
    assert rel(tr, want + (R0 if ef else 0)) <= (1e-6 if n % 4 else 1e-5)
    ref_codes, ref_scales = codec.quantize_transformed(tr, br, bc, shared)
    np.testing.assert_array_equal(scales, ref_scales)
    np.testing.assert_array_equal(codes, ref_codes)
    np.testing.assert_array_equal(scales2, ref_scales)
    np.testing.assert_array_equal(codes2, ref_codes)
    np.testing.assert_array_equal(hits.cpu().numpy().astype(np.int64), codec.boundary_hits(tr, codes))
    if ef:
        np.testing.assert_array_equal(R, codec.residual_after(tr, codes, scales, br, bc))
        np.testing.assert_array_equal(R2, R)
    mean = gpu_reduce(ctx, codes, scales, br, bc)
    np.testing.assert_array_equal(mean, codec.reduce_local(codes, scales, br, bc))
    if r:
        assert rel(gpu_decode(ctx, f, mean), codec.decode(mean, fA, fG)) <= 1e-6
        f.close()


@pytest.mark.parametrize("N,m,n,br,bc", [
    (1, 40, 259, 0, 0), (1, 17, 771, 5, 100), (2, 33, 1027, 0, 128), (2, 16, 254, 0, 7), (3, 31, 131, 0, 64),
    (3, 1500, 1503, 0, 128), (3, 1489, 1538, 7, 9), (4, 18, 67, 0, 0), (5, 18, 65, 0, 0),
])
def test_ragged_rank_sum(ctx, N, m, n, br, bc):  # noqa: F811
    """Few ranks take wide workgroups (256 columns), three of them from 512
    workgroups on: the mean bit for bit the oracle's."""
    say(f"ragged rank sum N={N} m={m} n={n} block=({br},{bc})")
    rng = np.random.default_rng(m + n)
    codes = rng.integers(0, 256, (N, m, n)).astype(np.uint8)
    codes[(codes & 0x7f) == 0x7f] = 0x38   # (no NaN)
    nbr, nbc = gift.scale_grid(m, n, br, bc)
    scales = rng.uniform(1e-6, 1e-3, (N, nbr, nbc)).astype(np.float32)
    mean = torch.full((m, n), float("nan"), device=DEV)
    gift.reduce_local(ctx, t(codes), t(scales), mean, br, bc)
    np.testing.assert_array_equal(mean.cpu().numpy(), codec.reduce_local(codes, scales, br, bc))
