"""Failure handling forced from the host: with KVX_FAULT=launch a call that
passes validation reports a failed launch (KVX_EHIP, hipErrorLaunchFailure)
and enqueues nothing, so the target cache keeps its previous contents; the
next call without the variable runs normally.  This is the path a runtime
takes to its fallback (native prefill) when a translation is unavailable.
No kernel is made to fail: the library returns before any launch.
Likewise the allocations of a fit (KVX_FAULT=fit-scratch, fit-solve) are
treated as refused without being tried.
"""
import os

import numpy as np
import pytest

from oracle import oracle as O
from paper_2608_30963_amd import kvx, synth as S
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

HIP_ERROR_LAUNCH_FAILURE = 719


@pytest.fixture
def fault_env():
    old = os.environ.get("KVX_FAULT")
    yield
    if old is None:
        os.environ.pop("KVX_FAULT", None)
    else:
        os.environ["KVX_FAULT"] = old


def _io(dev):
    prob, spec = dev.prob, dev.spec
    ident = prob.row_ptr is None
    return kvx.make_io(spec.batch, spec.src_tokens, dev.src_k, dev.src_v, dev.tgt_k, dev.tgt_v,
                       dev.cap, None if ident else prob.tgt_tokens, dev.row_ptr, dev.col_idx,
                       dev.weight)


def _untouched(dev):
    T = U.torch()
    T.cuda.synchronize()
    return bool(T.isnan(dev.tgt_k).all()) and bool(T.isnan(dev.tgt_v).all())


@pytest.mark.parametrize("cfg", [2, 3, 5])
def test_injected_launch_fault_then_recovery(cfg, fault_env):
    spec = S.config(cfg, src_tokens=260, batch=2)
    prob = S.make_problem(spec)
    print(f"[fault] {spec.name} KVX_FAULT=launch", flush=True)
    dev = U.DevProblem(prob)
    io, keep = _io(dev)
    os.environ["KVX_FAULT"] = "launch"
    st = kvx.kvx_translate_status(dev.tr.plan, io, U.torch().cuda.current_stream().cuda_stream)
    assert st == kvx.KVX_EHIP, kvx.status_string(st)
    assert kvx.load().kvx_last_hip_error() == HIP_ERROR_LAUNCH_FAILURE
    assert _untouched(dev), "a failed call wrote the target cache"
    # validation still comes first: a bad descriptor is reported as such
    bad, bkeep = kvx.make_io(spec.batch, spec.src_tokens, dev.src_k, dev.src_v, dev.tgt_k,
                             dev.tgt_v, 0, None if prob.row_ptr is None else prob.tgt_tokens,
                             dev.row_ptr, dev.col_idx, dev.weight)
    assert kvx.kvx_translate_status(dev.tr.plan, bad) != kvx.KVX_EHIP
    del bkeep
    # recovery: the same plan and buffers, without the fault
    del os.environ["KVX_FAULT"]
    print(f"[fault] {spec.name} recovery", flush=True)
    dev.run()
    U.torch().cuda.synchronize()
    rk, rv = O.translate(prob, cap=dev.cap)
    U.check_full(dev, rk, rv, f"after fault {spec.name}", 0.75)
    del keep
    dev.close()


def test_injected_launch_fault_staged(fault_env):
    T = U.torch()
    spec = S.config(2, src_tokens=260)
    prob = S.make_problem(spec)
    print("[fault] staged KVX_FAULT=launch", flush=True)
    dev = U.DevProblem(prob)
    io, keep = _io(dev)
    n = kvx.kvx_staged_workspace_bytes(dev.tr.plan, io, spec.tgt.n_layers)
    ws = T.empty(n, dtype=T.uint8, device="cuda")
    os.environ["KVX_FAULT"] = "launch"
    st = kvx.kvx_translate_staged_status(dev.tr.plan, io, ws.data_ptr(), n)
    assert st == kvx.KVX_EHIP, kvx.status_string(st)
    assert _untouched(dev)
    del os.environ["KVX_FAULT"]
    kvx.kvx_translate_staged(dev.tr.plan, io, ws)
    T.cuda.synchronize()
    rk, rv = O.translate(prob, cap=dev.cap)
    U.check_full(dev, rk, rv, "staged after fault", 0.75)
    del keep
    dev.close()


def _fit(layers, tokens, batch):
    """A fit of `layers` layers [512 -> 256] without bias (whose sums are
    atomic), and its drawn caches."""
    T = U.torch()
    g = T.Generator(device="cuda").manual_seed(5)
    draw = lambda *s: T.randn(s, generator=g, device="cuda").bfloat16()
    src, tgt = S.ModelShape(3, 4, 128, 1.0e6), S.ModelShape(layers, 2, 128, 1.0e6)
    x = [draw(3, batch, 4, tokens, 128) for _ in range(2)]
    y = [draw(layers, batch, 2, tokens, 128) for _ in range(2)]
    fit = kvx.Fitter(src, tgt, 1, [l % 3 for l in range(layers)], kvx.KVX_BF16, fit_bias=False)
    return fit, (x[0], x[1], y[0], y[1])


def test_fit_scratch_without_room_for_it(fault_env):
    """A device without room for a fit's scratch gets smaller groups of
    layers: 28 layers of 16384 rows in three of 1 GiB at most, to the same
    bits.  The limit stays with the fit."""
    fit, caches = _fit(28, 4096, 4)
    print("[fault] KVX_FAULT=fit-scratch", flush=True)
    fit.accumulate(*caches)
    want = fit.solve(1.0)
    fit.close()
    fit, caches = _fit(28, 4096, 4)
    held = fit.info().device_bytes
    os.environ["KVX_FAULT"] = "fit-scratch"
    fit.accumulate(*caches)
    del os.environ["KVX_FAULT"]
    assert 0 < fit.info().device_bytes - held <= 1 << 30
    fit.accumulate(*caches)
    assert fit.info().device_bytes - held <= 1 << 30
    fit.reset()
    fit.accumulate(*caches)
    for a, b in zip(fit.solve(1.0), want):
        assert U.torch().equal(a, b)
    fit.close()


def test_fit_solve_takes_the_scratch(fault_env):
    """A solve without room for its matrices releases the scratch of the
    accumulations and goes on; a fit without scratch reports KVX_ENOMEM, and
    works once there is room."""
    fit, caches = _fit(3, 200, 1)
    print("[fault] KVX_FAULT=fit-solve", flush=True)
    empty = fit.info().device_bytes
    os.environ["KVX_FAULT"] = "fit-solve"
    with pytest.raises(kvx.KvxError) as err:
        fit.solve(1.0)
    assert err.value.status == kvx.KVX_ENOMEM
    del os.environ["KVX_FAULT"]
    fit.accumulate(*caches)
    want = fit.solve(1.0)
    fit.close()
    fit, caches = _fit(3, 200, 1)
    fit.accumulate(*caches)
    assert fit.info().device_bytes > empty
    os.environ["KVX_FAULT"] = "fit-solve"
    got = fit.solve(1.0)
    del os.environ["KVX_FAULT"]
    solve_bytes = 6 * (512 * 512 + 512 * 256) * 8 + 256
    assert fit.info().device_bytes == empty + solve_bytes, "the scratch was kept"
    fit.accumulate(*caches)        # allocates its scratch again
    again = fit.solve(2.0)         # twice the rows, twice the ridge: the same weights
    for a, b, c in zip(got, want, again):
        assert U.torch().equal(a, b)
        U.torch().testing.assert_close(c, b, rtol=1e-4, atol=1e-5)
    fit.close()


def test_a_failed_plan_leaves_the_next_calls_alone():
    """A plan whose weights exceed the device's memory is refused with
    KVX_ENOMEM before its weights are read; the error ends with that call:
    the next plan is made, and a translation with it runs."""
    spec = S.config(2, src_tokens=40)
    prob = S.make_problem(spec)
    w = U.np_to_dev(prob.w_k, spec.dtype)
    big = S.ModelShape(1, 1024, 128, 1.0e4)   # 64 layers of [131072 -> 131072]: 4.4e12 bytes
    print("[fault] plan past the device's memory", flush=True)
    with pytest.raises(kvx.KvxError) as err:
        kvx.kvx_plan_create(big, S.ModelShape(64, 1024, 128, 1.0e4), 1, [0] * 64, kvx.KVX_BF16, w, w)
    assert err.value.status == kvx.KVX_ENOMEM
    dev = U.DevProblem(prob)
    dev.run()
    U.torch().cuda.synchronize()
    rk, rv = O.translate(prob, cap=dev.cap)
    U.check_full(dev, rk, rv, "after a failed plan", 0.75)
    dev.close()
