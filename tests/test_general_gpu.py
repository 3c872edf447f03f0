"""The general kernel (fp32 plans, and bf16 shapes the fused kernel does not
tile) at the edges of its tiles, against the oracle: 32-row tiles, chunks of
64 source pairs, groups of 4, 2 and 1 pair blocks of 32 outputs, whose waves
split the contraction when fewer than four.  A workgroup takes one pair block
while larger groups would leave compute units idle, so the long cases are the
ones that reach the groups."""
import pytest

from oracle import oracle as O
from paper_2608_30963_amd import synth as S

from . import gpu_util as G

pytestmark = pytest.mark.gpu

# (heads x dim) source, target, mix, tokens, batch, largest span, dtype
CASES = [
    ((1, 2), (1, 2), 1, 1, 1, 0, S.F32),        # smallest of everything
    ((2, 34), (3, 22), 1, 31, 2, 0, S.F32),     # 34 pairs (one chunk), 33 outputs (two blocks)
    ((3, 66), (1, 64), 2, 33, 1, 3, S.F32),     # 198 pairs: three chunks and a remainder
    ((1, 128), (2, 96), 1, 32, 3, 2, S.F32),    # three pair blocks
    ((2, 64), (7, 64), 1, 1029, 1, 0, S.F32),   # groups of 4, 2 and 1
    ((2, 64), (2, 64), 1, 1100, 2, 2, S.F32),   # a group of 2, spans
    ((3, 48), (5, 64), 1, 2050, 1, 0, S.F32),   # groups of 4 and 1
    ((8, 80), (4, 80), 1, 1057, 1, 2, S.BF16),  # groups of 4 and 1, bf16
    ((1, 10), (1, 18), 3, 65, 1, 4, S.BF16),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{c[1]}-x{c[2]}-{c[3]}-{c[6]}")
def test_general_kernel_tile_edges(case):
    (hs, ds), (ht, dt), mix, tokens, batch, span, dtype = case
    lt = 4
    lmap = tuple((l + j) % 5 for l in range(lt) for j in range(mix))
    spec = S.Spec(310, "general", S.ModelShape(5, hs, ds, 1.0e4), S.ModelShape(lt, ht, dt, 5.0e5),
                  mix, lmap, dtype, tokens, batch=batch, span_lo=1 if span else 0, span_hi=span,
                  bias_std=0.2)
    prob = S.make_problem(spec)
    dev = G.DevProblem(prob)
    assert dev.tr.info().kernel == 0
    dev.run()
    G.torch().cuda.synchronize()
    rk, rv = O.translate(prob)
    # bf16: correct rounding is 0.5 ulp, fp32 sums below it add under 0.01
    G.check_full(dev, rk, rv, "general", ulp_bound=0.6)
    dev.close()
