"""The encode's strip kernels (runs on an MI355X): the two passes of large
input-side encodes over column strips, at strips of 1 to 4 tile pairs, uneven
strips, ragged rows, few row groups per wave, block rows of one wave and with
the error-feedback residual; and launches just too small for strips.  Each case
states the strips that the kernels' own rule gives it, through a mirror of that
rule.

The reference is the same encode asked to store W~ (its block-maximum pass is
the per-unit kernel's): the codes, scales and residuals must be bit for bit
the quantization of that W~ by the oracle, checked on the first and last rank,
and the scales of every rank equal.
"""

import numpy as np
import pytest
import torch

from oracle import codec
from test_gpu_sweep import ctx, rel, say, t  # noqa: F401

pytestmark = pytest.mark.gpu

gift = pytest.importorskip("paper_2607_07494_amd.gift")
DEV = "cuda"


def strips_of(N, m, n, r, ef):
    """pick_strips of csrc/k_strip.hip: (strips per row chunk, 128-column tile
    pairs of the widest strip, strips that are one pair wider than the others),
    or None where the launch has too few 32-row groups for strips."""
    pairs, groups = n // 128, (m + 31) // 32 * N
    best, top = None, 0.0
    for s in range(1, 33):
        per = -(-pairs // s)
        chunks = 8 * (32 // s)
        rows = -(-groups // chunks)
        if per > (4 if r == 64 and not ef else 2) or s > pairs or rows < 16:
            continue
        use = pairs / (s * per) * groups / (chunks * 8 * -(-rows // 8))
        score = use * (chunks * s / 256) / (1 + 0.5 * r / (128 * per))
        if score > top:
            best, top = (s, per, pairs % s), score
    return best


@pytest.mark.parametrize("N,m,n,r,br,bc,ef,strips", [
    (30, 4100, 128, 64, 0, 128, False, (1, 1, 0)),     # one pair: one strip per row chunk, 256 chunks
    (2, 2000, 8192, 128, 0, 128, False, (32, 2, 0)),   # 32 strips of two pairs, eight chunks
    (4, 1500, 2816, 64, 0, 128, False, (22, 1, 0)),    # 22 pairs over the strips
    (5, 1201, 1664, 96, 0, 256, False, None),          # 13 pairs, blocks across them
    (8, 2016, 1152, 128, 32, 128, False, (9, 1, 0)),   # block rows of one row group
    (9, 3000, 1024, 64, 64, 0, False, (8, 1, 0)),      # whole rows in a block
    (3, 2500, 3072, 128, 0, 0, True, (24, 1, 0)),
    (6, 1999, 1024, 64, 0, 64, True, None),
    (4, 1999, 1536, 96, 0, 128, True, (12, 1, 0)),
    # strips of two to four pairs, some a pair narrower than the others
    (40, 1599, 384, 64, 0, 128, False, (2, 2, 1)),
    (40, 1599, 640, 64, 0, 64, False, (2, 3, 1)),
    (40, 1581, 896, 64, 64, 128, False, (2, 4, 1)),
    (20, 1599, 1664, 64, 0, 256, False, (4, 4, 1)),
    (40, 1599, 384, 64, 0, 128, True, (2, 2, 1)),
    (20, 1599, 896, 96, 0, 0, False, (4, 2, 3)),
    (20, 1570, 1152, 96, 32, 128, True, (5, 2, 4)),
    (40, 1599, 384, 128, 0, 256, False, (2, 2, 1)),
    (10, 1599, 1408, 128, 0, 64, True, (7, 2, 4)),
])
def test_strip_encode(ctx, N, m, n, r, br, bc, ef, strips):  # noqa: F811
    say(f"strip encode N={N} m={m} n={n} r={r} block=({br},{bc}) ef={ef} strips={strips}")
    assert strips_of(N, m, n, r, ef) == strips
    gen = torch.Generator(device=DEV)
    gen.manual_seed(m + n)
    U = np.linalg.qr(np.random.default_rng(n).standard_normal((n, r)))[0].astype(np.float32)
    c = np.linspace(-0.95, -0.3, r).astype(np.float32)
    f = gift.Factor(ctx, m, n, r, gift.SIDE_INPUT)
    f.import_(gift.SIDE_INPUT, t(U), t(c), t(-c), t(np.ones(1, np.float32)))
    g = torch.randn((N, m, n), generator=gen, device=DEV) * torch.randn((N, m, 1), generator=gen, device=DEV)
    R0 = torch.randn((N, m, n), generator=gen, device=DEV) * 0.01 if ef else None
    nbr, nbc = gift.scale_grid(m, n, br, bc)

    def encode(tr=None):
        codes = torch.full((N, m, n), 0x55, dtype=torch.uint8, device=DEV)
        scales = torch.full((N, nbr, nbc), float("nan"), device=DEV)
        R = R0.clone() if ef else None
        gift.encode(ctx, f, g, codes, scales, br, bc, gift.SCALE_LOCAL, ef=R, transformed=tr)
        return codes, scales, R

    tr = torch.empty((N, m, n), device=DEV)
    ref = encode(tr)
    for _ in range(2):   # the sub-slot sets alternate
        got = encode()
        torch.cuda.synchronize()
        for a, b in zip(got, ref):
            assert a is None or torch.equal(a, b)
    for j in sorted({0, N - 1}):
        W = g[j].double().cpu().numpy()
        want = W + (W @ U.astype(np.float64) * c) @ U.T.astype(np.float64)
        x = tr[j:j + 1].cpu().numpy()
        assert rel(x[0], want + (R0[j].cpu().numpy() if ef else 0)) <= 1e-5
        ref_codes, ref_scales = codec.quantize_transformed(x, br, bc, False)
        np.testing.assert_array_equal(got[1][j:j + 1].cpu().numpy(), ref_scales)
        np.testing.assert_array_equal(got[0][j:j + 1].cpu().numpy(), ref_codes)
        if ef:
            np.testing.assert_array_equal(got[2][j:j + 1].cpu().numpy(),
                                          codec.residual_after(x, ref_codes, ref_scales, br, bc))
    f.close()
