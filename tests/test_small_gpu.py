"""The small-call kernel (32-row tiles, segments of four chunks, two with
spans) and the persistent kernel on the same shapes, against the oracle and
against each other, bit for bit.  The call's size selects the kernel
(gpu_util.small_kernel), so the second batch size of each case is past the
line."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2608_30963_amd import kvx, synth as S

from . import gpu_util as G

pytestmark = pytest.mark.gpu

X2, F16, OUT = kvx.KVX_PREC_BF16X2, kvx.KVX_PREC_F16, kvx.KVX_PREC_BF16X2_OUTLIER
BF16 = kvx.KVX_PREC_BF16

# (heads x dim) source, target, mix, tokens, largest span, precision, small batch, large batch
CASES = [
    ((1, 128), (1, 64), 1, 1, 0, X2, 1, 60),     # smallest of everything
    ((4, 128), (2, 128), 1, 33, 0, X2, 2, 30),   # four chunks, one row past a tile
    ((4, 128), (2, 128), 1, 33, 0, F16, 2, 30),
    ((5, 128), (3, 128), 1, 31, 0, X2, 1, 30),   # a second segment of one chunk, half an N tile
    ((8, 128), (5, 64), 1, 64, 0, X2, 1, 15),    # two whole segments, two N tiles, the second of one block
    ((8, 32), (1, 256), 1, 40, 0, X2, 1, 30),    # four heads a chunk
    ((1, 256), (2, 128), 3, 65, 0, OUT, 1, 20),  # half a head a chunk, three mixed layers
    ((2, 64), (1, 128), 1, 70, 4, X2, 2, 60),    # spans past the two held entries
    ((3, 128), (4, 128), 1, 50, 2, X2, 1, 20),   # a second segment of one chunk, spans
    ((1, 256), (2, 512), 2, 90, 3, F16, 1, 10),  # angles afresh each chunk, spans
    ((8, 128), (2, 128), 1, 90, 3, X2, 1, 40),   # the interleaved order, spans
    ((2, 128), (4, 128), 1, 90, 5, X2, 1, 30),   # the resident order
    ((2, 64), (6, 64), 1, 60, 4, F16, 1, 30),    # the same with one chunk
    ((4, 128), (3, 128), 1, 40, 4, BF16, 2, 40),
]


@pytest.mark.parametrize("paged", [False, True], ids=["", "paged"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{c[1]}-x{c[2]}-{c[3]}-s{c[4]}-p{c[5]}")
def test_small_and_persistent_kernels(case, paged):
    (hs, ds), (ht, dt), mix, tokens, span, prec, small, large = case
    T = G.torch()
    lt = 5
    for batch in (small, large):
        spec = S.Spec(330, "small", S.ModelShape(4, hs, ds, 1.0e4), S.ModelShape(lt, ht, dt, 5.0e5),
                      mix, tuple((l + j) % 4 for l in range(lt) for j in range(mix)), S.BF16, tokens,
                      batch=batch, outliers=0 if prec in (F16, BF16) else 2, bias_std=0.3,
                      span_lo=1 if span else 0, span_hi=span)
        prob = S.make_problem(spec)
        marks = (S.outlier_channels(spec, 0), S.outlier_channels(spec, 1)) if prec == OUT else None
        cap = int(prob.tgt_tokens.max())
        dev = G.DevProblem(prob, prec, cap=cap, outliers=marks)
        assert dev.tr.info().kernel == 1
        assert G.small_kernel(prob, prec) == (batch == small)
        print(f"[small] {case} batch {batch} paged {paged}", flush=True)
        if paged:
            G.run_paged(dev)
        else:
            dev.run()
        T.cuda.synchronize()
        rk, rv = O.translate(prob, cap=cap)
        # split operands: 0.5 ulp of rounding and fp32 sums; else the operands'
        # own rounding, within check_close's envelope
        G.check_full(dev, rk, rv, f"batch {batch}", ulp_bound=0.75 if prec == X2 else None)
        gk = G.dev_to_f64(dev.tgt_k, spec.dtype)
        for b, t in enumerate(prob.tgt_tokens):
            assert np.isnan(gk[:, b, :, int(t):]).all(), "row past the context's end was written"
        dev.close()


@pytest.mark.parametrize("paged", [False, True], ids=["", "paged"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{c[1]}-x{c[2]}-{c[3]}-s{c[4]}-p{c[5]}")
def test_bits_do_not_depend_on_the_call(case, paged):
    """A context translated alone (the small kernel) and the same one in a
    batch (the persistent kernel, in each of its tile orders, into either
    layout) agree bit for bit."""
    (hs, ds), (ht, dt), mix, _, span, prec, _, _ = case
    T = G.torch()
    lt, tokens = 4, 200
    spec = S.Spec(331, "one-of-many", S.ModelShape(4, hs, ds, 1.0e4), S.ModelShape(lt, ht, dt, 5.0e5),
                  mix, tuple((l + j) % 4 for l in range(lt) for j in range(mix)), S.BF16, tokens,
                  batch=24, outliers=0 if prec in (F16, BF16) else 2, bias_std=0.3,
                  span_lo=1 if span else 0, span_hi=span)
    prob = S.make_problem(spec)
    marks = (S.outlier_channels(spec, 0), S.outlier_channels(spec, 1)) if prec == OUT else None
    cap = int(prob.tgt_tokens.max())
    dev = G.DevProblem(prob, prec, cap=cap, outliers=marks)
    n_cu = T.cuda.get_device_properties(0).multi_processor_count
    wgs = [-(-int(t) // 32) * -(-ht * dt // 256) * 2 * lt for t in prob.tgt_tokens]
    assert max(wgs) <= n_cu and not G.small_kernel(prob, prec), (wgs, n_cu)
    print(f"[small] {case} alone and in a batch, paged {paged}", flush=True)
    (G.run_paged if paged else G.DevProblem.run)(dev)
    first = 0
    for b in range(spec.batch):
        t = int(prob.tgt_tokens[b])
        one_k = T.full((lt, 1, ht, cap, dt), float("nan"), dtype=T.bfloat16, device="cuda")
        one_v = T.full_like(one_k, float("nan"))
        args = (None, None, None, None)
        if span:
            e0, e1 = int(prob.row_ptr[first]), int(prob.row_ptr[first + t])
            args = ([t], dev.row_ptr[first:first + t + 1] - e0, dev.col_idx[e0:e1].clone(),
                    dev.weight[e0:e1].clone())
        first += t
        dev.tr(dev.src_k[:, b:b + 1].contiguous(), dev.src_v[:, b:b + 1].contiguous(), one_k, one_v,
               cap, *args)
        for one, many in ((one_k, dev.tgt_k), (one_v, dev.tgt_v)):
            d = (one[:, 0, :, :t].view(T.int16) != many[:, b, :, :t].view(T.int16)).sum()
            assert int(d) == 0, f"context {b}: {int(d)} values differ"
    dev.close()
