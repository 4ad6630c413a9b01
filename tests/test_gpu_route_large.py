"""Routing and pruning of batches whose per-expert statistics come from their
own kernel, and of large ones whose do not.  SUM batches above 16 tokens always
take that kernel; under MAX and CIR lists of 12 or 16 from 33000 (token, slot)
pairs on, and lists of 8 from 16384 tokens on or where the tokens fill their
tiles of 4096 (the last one to 15/16).  Tokens in one, two and a partial third tile, lists whose rows are
16-byte aligned and not, one and several waves' worth of bins; every decision
equal to the oracle's, bin loads and sums bit for bit."""
import pytest
import torch

from caee_cases import check_route, gpu_layer, oracle_layer
from synth_inputs import TINY_F32, make_routing_inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
SHAPES = {4: TINY_F32.with_(name="k4", E=64, n_group=8, topk_group=4, k=4),
          6: TINY_F32.with_(name="k6", E=256, n_group=8, topk_group=4, k=6, bias_std=0.01),
          8: TINY_F32.with_(name="k8", E=128, n_group=4, topk_group=2, k=8),
          12: TINY_F32.with_(name="k12", E=256, n_group=4, topk_group=4, k=12),
          16: TINY_F32.with_(name="k16", E=48, n_group=3, topk_group=3, k=16)}


@pytest.mark.parametrize("rule,tau", [("max", 0.3), ("sum", 40.0), ("cir", 0.5)])
@pytest.mark.parametrize("k,T,n_bins", [
    (4, 4096, 32), (6, 4097, 1), (8, 2048, 4), (16, 1025, 8), (8, 9001, 32),
    # both sides of the line, MAX and CIR: with the kernel, then without
    (16, 2063, 8), (12, 2750, 1), (16, 4097, 1), (8, 4096, 1), (8, 12128, 32), (8, 16384, 4),
    (16, 2062, 8), (12, 2749, 32), (8, 12127, 1), (4, 10001, 1), (6, 7001, 32)])
def test_route_large(rule, tau, k, T, n_bins):
    shape = SHAPES[k]
    n_bins = n_bins if shape.E % n_bins == 0 else 1
    inp = make_routing_inputs(shape, seed=T, T=T, n_bins=n_bins, zipf_logit_s=1.1, cost_kind="zipf")
    print(f"route k={k} T={T} {rule} bins={n_bins}", flush=True)
    got = gpu_layer(shape, inp, tau, n_bins, None, DEV, route_only=True, rule=rule)
    ref = oracle_layer(shape, inp, tau, n_bins, with_y=False, rule=rule)
    check_route(got, ref, shape.E)


@pytest.mark.parametrize("T", [17, 63, 64, 65, 300])
def test_route_sum_small_batches(T):
    shape = SHAPES[8]
    inp = make_routing_inputs(shape, seed=T, T=T, n_bins=4, zipf_logit_s=1.1, cost_kind="zipf")
    got = gpu_layer(shape, inp, 1.2, 4, None, DEV, route_only=True, rule="sum")
    check_route(got, oracle_layer(shape, inp, 1.2, 4, with_y=False, rule="sum"), shape.E)
