"""The general kernel (fp32 plans, and bf16 shapes the fused kernel does not
tile) at the edges of its tiles, against the oracle: 32-row tiles, chunks of
64 source pairs, groups of 4, 2 and 1 pair blocks of 32 outputs, whose waves
split the contraction when fewer than four.  A workgroup takes one pair block
while larger groups would leave compute units idle, so the long cases are the
ones that reach the groups."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_2608_30963_amd import kvx, synth as S

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

# products that the row kernel takes, whatever the rows or for few (fp32: under
# 1024 values, or 2304; bf16: 3072, 6400, or 8192 at 8 source pairs), and the
# first one past each
ROW_CASES = [
    ((1, 2), (1, 2), 1, 17, 2, 0, S.F32),
    ((1, 22), (1, 46), 1, 2100, 1, 2, S.F32),     # 1012: whatever the rows
    ((1, 32), (1, 32), 1, 2100, 1, 0, S.F32),     # 1024: not for many rows
    ((1, 48), (2, 24), 1, 1024, 1, 3, S.F32),     # 2304
    ((1, 48), (1, 50), 1, 33, 1, 0, S.F32),
    ((1, 16), (2, 40), 1, 2100, 1, 0, S.F32),     # 1280 of 8 source pairs
    ((2, 16), (3, 32), 1, 2100, 1, 2, S.BF16),    # 3072
    ((1, 80), (1, 80), 1, 1024, 1, 0, S.BF16),    # 6400
    ((1, 80), (1, 82), 1, 1024, 1, 2, S.BF16),
    ((1, 16), (4, 128), 1, 1100, 2, 0, S.BF16),   # 8192 of 8 source pairs
    ((3, 8), (1, 10), 2, 5, 66, 2, S.BF16),       # short contexts, two launches
]


@pytest.mark.parametrize("case", CASES + ROW_CASES, ids=lambda c: f"{c[0]}-{c[1]}-x{c[2]}-{c[3]}-{c[6]}")
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


@pytest.mark.parametrize("paged", [False, True], ids=["", "paged"])
@pytest.mark.parametrize("dtype,tokens,batch,lengths", [
    (S.F32, 1, 70, None),              # one row each; a second launch of six contexts
    (S.BF16, 3, 67, None),
    (S.F32, 40, 9, [0, 1, 0, 40, 5, 0, 31, 33, 0]),   # empty ones first, between and last
    (S.BF16, 9, 66, [0] * 64 + [9, 2]),               # a launch without rows, then one with
])
def test_general_kernel_contexts_share_tiles(dtype, tokens, batch, lengths, paged):
    """Tiles that hold the rows of several contexts, whole or in part."""
    T = G.torch()
    spec = S.Spec(312, "shared-tiles", S.ModelShape(4, 2, 40, 1.0e4), S.ModelShape(3, 3, 24, 5.0e5),
                  1, (3, 0, 2), dtype, tokens, batch=batch, bias_std=0.2,
                  span_lo=1 if lengths else 0, span_hi=2 if lengths else 0)
    prob = S.make_problem(spec)
    if lengths:
        rng = np.random.default_rng(7)
        n = rng.integers(0, 4, size=sum(lengths))
        prob = dataclasses.replace(
            prob, tgt_tokens=np.array(lengths, dtype=np.int32),
            row_ptr=np.concatenate([[0], np.cumsum(n)]).astype(np.int32),
            col_idx=rng.integers(0, tokens, size=int(n.sum())).astype(np.int32),
            weight=rng.uniform(-1.0, 1.0, size=int(n.sum())).astype(np.float32))
    cap = int(prob.tgt_tokens.max())
    dev = G.DevProblem(prob, cap=cap)
    assert dev.tr.info().kernel == 0
    print(f"[general] {tokens} x {batch} paged {paged}", flush=True)
    (G.run_paged if paged else G.DevProblem.run)(dev)
    T.cuda.synchronize()
    rk, rv = O.translate(prob, cap=cap)
    G.check_full(dev, rk, rv, "shared tiles", ulp_bound=0.6)
    gk = G.dev_to_f64(dev.tgt_k, spec.dtype)
    for b, t in enumerate(prob.tgt_tokens):
        assert np.isnan(gk[:, b, :, int(t):]).all(), "row past the context's end was written"
    dev.close()


@pytest.mark.parametrize("dtype,prec", [(S.F32, kvx.KVX_PREC_BF16X2), (S.BF16, kvx.KVX_PREC_BF16X2),
                                        (S.BF16, kvx.KVX_PREC_F16)])
def test_plan_weights_by_memory_kind(dtype, prec):
    """Weights in pinned host memory give the plan that device weights give;
    pageable host memory, and device memory that ends before the weights do,
    are refused on the host."""
    T = G.torch()
    spec = S.Spec(311, "weights", S.ModelShape(2, 2, 128, 1.0e4), S.ModelShape(2, 1, 128, 5.0e5),
                  1, (1, 0), dtype, 70, batch=1, bias_std=0.2)
    prob = S.make_problem(spec)
    dev = G.DevProblem(prob, prec)
    dev.run()
    want_k, want_v = dev.tgt_k.clone(), dev.tgt_v.clone()
    host = [w.cpu() for w in (dev.w_k, dev.w_v)]

    def plan(w_k, w_v):
        return kvx.Translator(spec.src, spec.tgt, spec.mix, spec.layer_map, dev.kdtype, w_k, w_v,
                              dev.b_k, dev.b_v, precision=prec)
    dev.tr.close()
    dev.tr = plan(host[0].pin_memory(), host[1].pin_memory())
    dev.tgt_k.fill_(0)
    dev.tgt_v.fill_(0)
    dev.run()
    T.cuda.synchronize()
    assert T.equal(dev.tgt_k, want_k) and T.equal(dev.tgt_v, want_v)
    nbytes = host[0].numel() * host[0].element_size()
    T.cuda.empty_cache()
    block = T.empty(64 << 20, dtype=T.uint8, device="cuda")   # an allocation of its own
    end = block.data_ptr() + block.numel()
    for bad_k, bad_v in ((host[0], dev.w_v), (dev.w_k, host[1]), (dev.w_k, end - nbytes + 16)):
        with pytest.raises(kvx.KvxError) as err:
            plan(bad_k, bad_v)
        assert err.value.status == kvx.KVX_EHIP
    dev.close()
