"""GPU factor statistics A = X^T X / T against the oracle (runs on an MI355X).

Step a1 of the hot path (eq. kfac_fisher_block, eq. impl_A_psd), called
through ``gift_statistics``.  bfloat16 inputs with dim % 8 == 0 run on the
bf16 SYRK kernel (256 x 256 tiles, 64-token stages); other inputs on the
float32 tile kernel.  Shapes span several tiles with ragged feature and token
tails, single-stage and sub-stage token counts, and the widening path.

Bars, both checked element by element against the float64 oracle:
* the rigorous float32 summation bound |A_gpu - A| <= (gamma_T + u) |X|^T |X| / T
  with u = 2^-24, gamma_T = T u / (1 - T u) (every product of two bf16 values
  is exact in float32; only the T-term sums and the 1/T scale round);
* relative Frobenius error <= 5e-6 (blocked float32 accumulation over at most
  a few thousand terms, about sqrt(T/32) u).
"""

import numpy as np
import pytest
import torch

from oracle import codec
from synth import factor_inputs

pytestmark = pytest.mark.gpu

gift = pytest.importorskip("paper_2607_07494_amd.gift")
DEV = "cuda"
U32 = 2.0 ** -24


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = gift.Context()
    yield c
    torch.cuda.synchronize()
    c.close()


def device_input(T, dim, dtype, seed):
    x, bits = factor_inputs(seed, T, dim, dtype=dtype)
    if dtype == "bf16":
        xt = torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).to(DEV)
    else:
        xt = torch.from_numpy(x).to(DEV)
    return x, xt


CASES = [
    # (T, dim, dtype)
    (1000, 72, "bf16"),     # one partial tile, ragged last stage
    (4160, 520, "bf16"),    # 3 x 3 tiles (6 computed), tail of 8 features
    (2048, 256, "bf16"),    # exactly one tile
    (64, 1032, "bf16"),     # one token stage, 5 x 5 tiles
    (37, 24, "bf16"),       # fewer tokens than one stage
    (3001, 776, "bf16"),    # odd T, 4 x 4 tiles
    (300, 50, "bf16"),      # dim % 8 != 0: widened to float32, tile kernel
    (1500, 130, "f32"),     # float32 tile kernel
]


@pytest.mark.parametrize("T,dim,dtype", CASES)
def test_statistics_match_oracle(ctx, T, dim, dtype):
    say(f"statistics T={T} dim={dim} dtype={dtype}")
    x, xt = device_input(T, dim, dtype, seed=7000 + dim)
    A = torch.full((dim, dim), float("nan"), dtype=torch.float32, device=DEV)
    gift.statistics(ctx, xt, A)
    torch.cuda.synchronize()
    got = A.cpu().numpy().astype(np.float64)
    ref = codec.factor_statistics(x)
    assert np.all(np.isfinite(got)), "unwritten or non-finite entries"
    ax = np.abs(x.astype(np.float64))
    bound = (T * U32 / (1 - T * U32) + U32) * (ax.T @ ax) / T + 1e-30
    err = np.abs(got - ref)
    worst = float(np.max(err / bound))
    assert worst <= 1.0, f"summation bound exceeded by {worst:.2f}x"
    rel = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    assert rel <= 5e-6, f"relative Frobenius error {rel:.2e}"
    asym = float(np.max(np.abs(got - got.T)) / np.max(np.abs(ref)))
    assert asym <= 1e-6


def test_statistics_repeat_is_deterministic(ctx):
    say("statistics determinism")
    _, xt = device_input(2500, 600, "bf16", seed=7100)
    A1 = torch.empty((600, 600), dtype=torch.float32, device=DEV)
    A2 = torch.empty_like(A1)
    gift.statistics(ctx, xt, A1)
    gift.statistics(ctx, xt, A2)
    torch.cuda.synchronize()
    assert torch.equal(A1, A2)


def test_refresh_of_many_dimensions(ctx):
    """Ten input dimensions in one refresh, more than one launch of the bf16
    statistics takes, a dimension outside that kernel among them: the tiles are
    those of a refresh alone, so the factors are too."""
    say("statistics of many dimensions")
    T, r = 96, 4
    dims = [8, 264, 16, 300, 24, 256, 40, 520, 72, 104]
    acts = [device_input(T, d, "bf16" if d != 300 else "f32", seed=7200 + d)[1].to(torch.bfloat16) for d in dims]
    batch = [gift.Factor(ctx, 8, d, r, gift.SIDE_INPUT, seed=d) for d in dims]
    gift.factor_update_batch(ctx, batch, acts, [None] * len(dims), iters=2)
    for d, x, f in zip(dims, acts, batch):
        one = gift.Factor(ctx, 8, d, r, gift.SIDE_INPUT, seed=d)
        one.update(acts=x, iters=2)
        for a, b in zip(f.export(gift.SIDE_INPUT), one.export(gift.SIDE_INPUT)):
            if isinstance(a, torch.Tensor):
                assert torch.equal(a, b), d
            else:
                assert a == b, d
        one.close()
        f.close()


def test_statistics_argument_errors(ctx):
    say("statistics errors")
    x = torch.zeros((16, 8), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(ValueError):
        gift.statistics(ctx, x, torch.zeros((4, 4), dtype=torch.float32, device=DEV))
    with pytest.raises(TypeError):
        gift.statistics(ctx, x.to(torch.float16), torch.zeros((8, 8), dtype=torch.float32, device=DEV))
