"""GPU parity at the sizes where the FFN's dispatch changes: the batch from
which the 8-bit big chunks take the prefill kernel, the mean rows per expert
from which every chunk is a big one (and the small-chunk kernels are not
launched), and the shapes and layouts those rules leave to the other kernels.
Tolerances are those of the tiny-layer tests of each type."""
import pytest
import torch

from caee_cases import check_route, check_y, getters_np, gpu_layer, oracle_layer, to_dev, w_to_dev
from paper_2606_29982_amd import caee
from synth_inputs import TINY_F32, make_expert_weights_np, make_expert_weights_torch, make_routing_inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
FP8 = TINY_F32.with_(name="tiny-fp8", w_dtype="fp8", x_dtype="bf16", y_dtype="bf16")
BF16 = TINY_F32.with_(name="tiny-bf16", w_dtype="bf16", x_dtype="bf16", y_dtype="bf16")
# 64 experts, 4 per token: 8 rows per expert at 128 tokens; 48 experts in 3
# groups, none shared: an expert count that is no power of two
WIDE8 = FP8.with_(name="wide-fp8", E=64, n_group=8, topk_group=4)
ODD8 = FP8.with_(name="odd-fp8", E=48, n_group=3, topk_group=2, n_shared=0)
# 384 is no multiple of 256: the staged kernels take the big chunks
D384 = FP8.with_(name="fp8-384", d=384, E=64, n_group=8, topk_group=4)


def _case(shape, T, tiled=True, zipf=1.1, tol=None):
    inp = make_routing_inputs(shape, seed=T, T=T, n_bins=1, zipf_logit_s=zipf)
    W = make_expert_weights_np(shape, seed=5)
    Wd = w_to_dev(W, DEV)
    if tiled:
        Wd = caee.pack_weights(Wd, shape.w_dtype)
    print(f"{shape.name} T={T} tiled={tiled} zipf={zipf}", flush=True)
    got = gpu_layer(shape, inp, 0.0, 1, Wd, DEV)
    get, get_sh = getters_np(W, shape.w_dtype)
    ref = oracle_layer(shape, inp, 0.0, 1, get, get_sh)
    check_route(got, ref, shape.E)
    check_y(got["y"], ref["y"], tol or {"fp8": 6e-2, "bf16": 2e-2}[shape.w_dtype])


@pytest.mark.parametrize("shape", [WIDE8, ODD8])
@pytest.mark.parametrize("T", [32, 33, 95, 96, 127, 128, 257])
@pytest.mark.parametrize("zipf", [None, 1.1])
def test_fp8_rules(shape, T, zipf):
    _case(shape, T, zipf=zipf)


# Up to 16 tokens the routing launch quantises x, up to 4 it runs the shared
# experts' gate/up; contractions of 2, 9, 20 and 65 blocks of 128 over its 16
# waves (idle waves, several blocks a wave, more than four).
@pytest.mark.parametrize("d,n_shared,tiled", [(256, 1, True), (1152, 2, False), (2560, 0, True), (8320, 1, True)])
@pytest.mark.parametrize("T", [1, 3, 4, 5, 16, 17])
def test_fp8_small_batches(d, n_shared, tiled, T):
    _case(FP8.with_(name=f"fp8-small-{d}", d=d, f=256, E=8, n_group=2, topk_group=1, k=3, n_shared=n_shared), T,
          tiled=tiled, zipf=None)


@pytest.mark.parametrize("shape,tiled", [(D384, True), (WIDE8, False)])
@pytest.mark.parametrize("T", [33, 130, 300])
def test_fp8_staged(shape, tiled, T):
    _case(shape, T, tiled=tiled)


@pytest.mark.parametrize("tiled", [True, False])
@pytest.mark.parametrize("T", [55, 56, 200])
def test_bf16_rules(T, tiled):
    # 16 experts, 4 per token: 14 rows per expert at 56 tokens
    _case(BF16, T, tiled=tiled)


# Which chunk list stays on the main stream: the small one without shared
# experts, until the routed experts have 12 rows each (48 tokens here); the big
# one with them.  Popular experts, so that both lists hold chunks; row-major and
# d = 384 as well, whose big chunks other kernels take.
@pytest.mark.parametrize("shape", [TINY_F32, BF16, FP8])
@pytest.mark.parametrize("n_shared,T", [(0, 33), (0, 47), (0, 48), (2, 47)])
@pytest.mark.parametrize("d,tiled", [(256, True), (384, True), (256, False)])
def test_list_order(shape, n_shared, T, d, tiled):
    _case(shape.with_(name=f"order-{shape.w_dtype}-{d}-{n_shared}", d=d, n_shared=n_shared), T, tiled=tiled,
          tol=1e-5 if shape.w_dtype == "f32" else None)


# Contractions whose stage counts leave 1, 2 and 3 steps after the stage loop
# (bf16: 64-element stages; 8-bit: 128), every token-tile count, experts in one
# chunk and in several (whose weights take the cached loads), odd tile counts
# among them; d = 384 goes to the staged kernels.
@pytest.mark.parametrize("d,f", [(1280, 128), (256, 384), (512, 1408), (384, 256)])
@pytest.mark.parametrize("T,zipf", [(100, None), (300, 1.1), (600, None), (777, 1.1)])
def test_bf16_gemm(d, f, T, zipf):
    _case(BF16.with_(name=f"bf16-{d}-{f}", d=d, f=f), T, zipf=zipf)


@pytest.mark.parametrize("d,f", [(1280, 384), (768, 640), (256, 896)])
@pytest.mark.parametrize("T,zipf", [(300, 1.1), (1300, None), (1500, 1.1)])
def test_fp8_prefill_tails(d, f, T, zipf):
    _case(FP8.with_(name=f"fp8-{d}-{f}", d=d, f=f), T, zipf=zipf)


def test_noalloc_limit_of_decode_batches():
    # The transposed block scales do not count against the scratch limit: the
    # largest 8-bit batch under it runs and equals the call with a workspace,
    # the next one is refused.
    shape = FP8.with_(name="noalloc-fp8", d=8192, f=256, k=8, n_shared=4)

    def counted(T):
        layer = caee.Layer.from_shape(shape, T=T, tau=0.0, n_bins=1)
        rows = T * (shape.k + shape.n_shared)
        pad = lambda n: (n + 255) & ~255  # noqa: E731
        return layer, caee.workspace_size(layer) - pad(rows * shape.d // 32) - pad(rows * shape.f // 32)

    T = max(t for t in range(33, 257) if counted(t)[1] <= caee.SCRATCH_BYTES)
    assert T < 256 and caee.workspace_size(counted(T)[0]) > caee.SCRATCH_BYTES
    Wd = caee.pack_weights(make_expert_weights_torch(shape, seed=6, device=DEV), "fp8")
    for t, fits in ((T, True), (T + 1, False)):
        layer = counted(t)[0]
        inp = make_routing_inputs(shape, seed=7, T=t, n_bins=1)
        a = (to_dev(inp.x, DEV), to_dev(inp.logits, DEV), None, to_dev(inp.cost, DEV), None, Wd)
        ya, yb = (torch.full((t, shape.d), 5.0, dtype=torch.bfloat16, device=DEV) for _ in range(2))
        print(f"noalloc fp8 T={t} fits={fits}", flush=True)
        if fits:
            caee.moe_layer(layer, *a, ya, caee.alloc_workspace(layer, DEV))
            caee.moe_layer_noalloc(layer, *a, yb)
            torch.cuda.synchronize()
            assert torch.equal(ya, yb)
        else:
            with pytest.raises(caee.CaeeError) as ei:
                caee.moe_layer_noalloc(layer, *a, yb)
            assert ei.value.status == caee.CAEE_ERR_UNSUPPORTED
