"""bench.py's figures of the products of a classifier's step: every call that multiplies is timed, labelled and counted once, the calls
that hold a layer's whole backward among them."""
import os
import sys
import time

import pytest
import torch

from paper_1908_00213_amd import workloads as W

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


@pytest.mark.parametrize("in_one_call", [(False, False, False), (True, True, True), (True, False, True)])
def test_the_calls_hold_the_operations_of_the_step(in_one_call):
    w = W.config1()
    calls = bench.gemm_calls_mlp(w.sizes, w.batch, False, in_one_call)
    assert len(calls) == 8 - sum(in_one_call[1:])
    res = bench.gemm_report(calls, [2e-6] * len(calls), 1e-6)
    assert res["gemm_flops_per_step"] == w.flops_per_step() and abs(res["gemm_seconds_per_step"] - 2e-6 * len(calls)) < 1e-12
    assert [c["call"] for c in res["gemm_calls"]] == [lab for lab, _ in calls]


def test_times_without_a_label_are_refused():
    w = W.config1()
    calls = bench.gemm_calls_mlp(w.sizes, w.batch, False, (False, False, False))
    with pytest.raises(RuntimeError):
        bench.gemm_report(calls, [1e-6] * 3, 0.0)


class _Once:
    def repeats(self, fn, steps, warmup, repeats):
        fn()
        torch.cuda.synchronize()
        t = time.perf_counter()
        fn()
        torch.cuda.synchronize()
        return [time.perf_counter() - t] * repeats


@pytest.mark.gpu
@pytest.mark.parametrize("fused_update", [False, True])
@pytest.mark.parametrize("workload", ["tiny", "wide"])
def test_every_product_of_a_recorded_step_is_timed(workload, fused_update):
    from paper_1908_00213_amd import binding as B, steps
    w = W.config1() if workload == "tiny" else W.config5(n_batches=1, scale=8)      # (the wide one: bias gradients out of the input gradients' products)
    r = bench.bench_mlp(torch, B, steps, w, workload == "wide", _Once(), 1, 1, probe=True, fused_update=fused_update, probe_steps=2)
    assert r["gemm_flops_per_step"] == w.flops_per_step()
    assert all(c["us"] > 0 for c in r["gemm_calls"])
    assert abs(sum(c["us"] for c in r["gemm_calls"]) * 1e-6 - r["gemm_seconds_per_step"]) < 1e-7 * len(r["gemm_calls"])
