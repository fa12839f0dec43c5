"""The encode's strip kernels (runs on an MI355X): the two passes of large
input-side encodes over column strips, at strips of 1 to 4 tile pairs, uneven
strips, ragged rows, few row groups per wave, block rows of one wave and with
the error-feedback residual; and launches for which strips are too few or not
the faster ones, in one pass or both.  Each case states the strips that the
kernels' own rule gives it, through a mirror of that rule.

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
    """pick_strips and lr_strip_eligible of csrc/k_strip.hip: (strips per row
    chunk, 128-column tile pairs of the widest strip, strips that are one pair
    wider than the others, the passes that take them), or None where neither
    does."""
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
    if best is None or not ef:
        return best and best + ("maxima codes",)
    fill = pairs * 8 * (32 // best[0]) / (256 * best[1])
    passes = []
    if fill >= 0.8:
        passes.append("maxima")
    large = 4 * N * m * n > 224 << 20 and (r < 128 or fill < 0.85)
    if (fill >= 0.8 and not large) or (r == 64 and n % 256):
        passes.append("codes")
    return best + (" ".join(passes),) if passes else None


BOTH = "maxima codes"


@pytest.mark.parametrize("N,m,n,r,br,bc,ef,strips", [
    (30, 4100, 128, 64, 0, 128, False, (1, 1, 0, BOTH)),     # one pair: one strip per row chunk, 256 chunks
    (2, 2000, 8192, 128, 0, 128, False, (32, 2, 0, BOTH)),   # 32 strips of two pairs, eight chunks
    (4, 1500, 2816, 64, 0, 128, False, (22, 1, 0, BOTH)),    # 22 pairs over the strips
    (5, 1201, 1664, 96, 0, 256, False, None),                # 13 pairs, blocks across them
    (8, 2016, 1152, 128, 32, 128, False, (9, 1, 0, BOTH)),   # block rows of one row group
    (9, 3000, 1024, 64, 64, 0, False, (8, 1, 0, BOTH)),      # whole rows in a block
    # (a quarter of the chip idle: not with the residual)
    (3, 2500, 3072, 128, 0, 0, True, None),
    (6, 1999, 1024, 64, 0, 64, True, None),
    (4, 1999, 1536, 96, 0, 128, True, None),
    # strips of two to four pairs, some a pair narrower than the others
    (40, 1599, 384, 64, 0, 128, False, (2, 2, 1, BOTH)),
    (40, 1599, 640, 64, 0, 64, False, (2, 3, 1, BOTH)),
    (40, 1581, 896, 64, 64, 128, False, (2, 4, 1, BOTH)),
    (20, 1599, 1664, 64, 0, 256, False, (4, 4, 1, BOTH)),
    (20, 1599, 896, 96, 0, 0, False, (4, 2, 3, BOTH)),
    (40, 1599, 384, 128, 0, 256, False, (2, 2, 1, BOTH)),
    # with the residual
    (7, 1599, 2048, 128, 0, 0, True, (16, 1, 0, BOTH)),
    (20, 1570, 1152, 64, 0, 64, True, (5, 2, 4, BOTH)),
    (20, 1570, 1152, 96, 32, 128, True, (5, 2, 4, BOTH)),
    (20, 1599, 1152, 128, 0, 128, True, (5, 2, 4, BOTH)),
    (9, 1599, 1664, 128, 0, 128, True, (13, 1, 0, BOTH)),
    # (one pass strips, the other the sweep or the per-unit kernel)
    (40, 1599, 384, 64, 0, 128, True, (2, 2, 1, "codes")),
    (40, 1599, 1024, 96, 0, 128, True, (4, 2, 0, "maxima")),
    (10, 1599, 1408, 128, 0, 64, True, None),
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
