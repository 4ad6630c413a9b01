"""GPU parity of the 8-bit expert path: OCP e4m3 weights with fp32 128x128
block scales, activations quantised per token per 128 channels.  Indices
exact, outputs within 6e-2 * max|ref| of the fp64 oracle (which quantises
the same activations the same way)."""
import numpy as np
import pytest
import torch

from caee_cases import check_route, check_y, getters_dev, getters_np, gpu_layer, oracle_layer, w_to_dev
from paper_2606_29982_amd import caee
from synth_inputs import R1_FP8, TINY_F32, make_expert_weights_np, make_expert_weights_torch, make_routing_inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
TINY_FP8 = TINY_F32.with_(name="tiny-fp8", w_dtype="fp8", x_dtype="bf16", y_dtype="bf16")


def _tiny(seed, tau, n_bins, T=None, rule="max", tiled=False, zipf=None, shape=TINY_FP8):
    inp = make_routing_inputs(shape, seed=seed, T=T, n_bins=n_bins, zipf_logit_s=zipf)
    W = make_expert_weights_np(shape, seed=seed)
    Wd = w_to_dev(W, DEV)
    if tiled:
        Wd = caee.pack_weights(Wd, "fp8")
    print(f"fp8 tiny seed={seed} tau={tau} n_bins={n_bins} T={inp.logits.shape[0]} rule={rule} tiled={tiled}",
          flush=True)
    got = gpu_layer(shape, inp, tau, n_bins, Wd, DEV, rule=rule)
    get, get_sh = getters_np(W, "fp8")
    ref = oracle_layer(shape, inp, tau, n_bins, get, get_sh, rule=rule)
    check_route(got, ref, shape.E)
    return check_y(got["y"], ref["y"], 6e-2)


@pytest.mark.parametrize("seed", range(3))
@pytest.mark.parametrize("tiled", [False, True])
def test_tiny_fp8(seed, tiled):
    rel = _tiny(seed, 0.1, 4, tiled=tiled)
    print(f"  max|err|/max|ref| = {rel:.3e}")


# 20 and 70 tokens: the shared expert's rows in the small and in the big
# list.  T=600 and 1100 take the prefill GEMM (128-row chunks; down runs the
# pairs of chunks of an expert cut into several in its 128 x 256 shape, and a
# last odd chunk alone): ragged chunk tails, a one-block contraction in the
# down product (f=128) and two in gate/up.
@pytest.mark.parametrize("T", [1, 5, 20, 40, 70, 130, 600, 1100])
def test_tiny_fp8_batches(T):
    _tiny(7, 0.2, 4, T=T, tiled=True, zipf=1.1 if T > 100 else None)


# d = f = 1024: both contractions are multiples of four 128-deep blocks, so
# down items may run several weight groups of a chunk back to back (8 gate/up
# groups of 128 features, 4 down groups of 256 rows).  d = 1280: five down
# groups.  These batches have too few chunks for that (test_fp8_down_runs below
# has enough): their items are single groups.
# 400 tokens: routed chunks of about 100 rows (7 token tiles) and the shared
# expert's 400 rows in two chunks of 200 (13 tiles); every output compared.
MID_FP8 = TINY_FP8.with_(name="mid-fp8", d=1024, f=1024)
MID_FP8_5 = TINY_FP8.with_(name="mid-fp8-5", d=1280, f=1024)


@pytest.mark.parametrize("seed,shape", [(11, MID_FP8), (12, MID_FP8), (13, MID_FP8_5)])
def test_mid_fp8_prefill(seed, shape):
    rel = _tiny(seed, 0.1, 4, T=400, tiled=True, shape=shape)
    print(f"  {shape.name}: max|err|/max|ref| = {rel:.3e}")


# Down items of four groups (129 chunks of 5 groups, so a chunk's last run is a
# single group) and of two (129 chunks of 4 groups), which an MI355X's 256 CUs
# take at 200 tokens over 128 experts and the shared one; 60 tokens leave the
# experts without eight rows each in the small list and the runs at one group.
@pytest.mark.parametrize("d,T", [(1280, 200), (1024, 200), (1280, 60)])
def test_fp8_down_runs(d, T):
    shape = TINY_FP8.with_(name=f"runs-fp8-{d}", d=d, f=512, E=128, n_group=4, topk_group=4, k=8)
    W = make_expert_weights_torch(shape, seed=2, device=DEV)
    inp = make_routing_inputs(shape, seed=2, T=T, n_bins=4)
    print(f"fp8 down runs d={d} T={T}", flush=True)
    got = gpu_layer(shape, inp, 0.0, 4, caee.pack_weights(W, "fp8"), DEV)
    tokens = list(range(0, T, 9))
    get, get_sh = getters_dev(W, "fp8")
    ref = oracle_layer(shape, inp, 0.0, 4, get, get_sh, tokens=tokens)
    check_route(got, ref, shape.E)
    if T == 200:
        assert ref["stats"]["n_act"] == 128
    check_y(got["y"][tokens], ref["y"], 6e-2)


def test_tiny_fp8_sum_rule():
    _tiny(8, 0.8, 4, rule="sum", tiled=True)


def test_e4m3_codes_match_oracle():
    # the activation codec: quantise rows whose values hit every rounding
    # case (ties, subnormals, the saturation edge) and compare the dequantised
    # rows with the oracle's fp32 quantiser
    from oracle import quantize_e4m3_blocks
    rng = np.random.default_rng(0)
    rows = rng.standard_normal((64, 256)).astype(np.float32) * np.float32(3.0)
    rows[0, :128] = np.linspace(-448, 448, 128, dtype=np.float32)
    rows[1, :128] = 2.0 ** -np.arange(128, dtype=np.float32) * 0.5
    rows[2, :] = 0.0
    # every tie of the codec: 448 (so the block scale is exactly 1) and the
    # midpoint between each pair of consecutive codes, both signs; the
    # midpoints have 5 significant bits, so the bf16 rows hold them exactly
    from oracle import e4m3_decode as _dec
    vals = _dec(np.arange(127, dtype=np.uint8))
    ties = np.concatenate([[448.0], (vals[:-1] + vals[1:]) / 2, [vals[1] / 4]]).astype(np.float32)
    rows[3, :128] = ties
    rows[3, 128:] = -ties
    import synth_inputs
    bits = synth_inputs.bf16_bits_from_f32(rows)
    x = torch.from_numpy(bits.view(np.int16)).to(DEV).view(torch.bfloat16)
    exact = (bits.astype(np.uint32) << 16).view(np.float32)
    _, scale_ref, deq_ref = quantize_e4m3_blocks(exact)
    # run the quantiser through a 1-token-per-row layer: compare via a layer
    # whose experts are identity-like is indirect, so call the path directly
    T, d = rows.shape
    q = torch.empty((T, d), dtype=torch.uint8, device=DEV)
    s = torch.empty((T, d // 128), dtype=torch.float32, device=DEV)
    caee.quantize_rows(x, q, s)
    torch.cuda.synchronize()
    from oracle import e4m3_decode
    deq = e4m3_decode(q.cpu().numpy()).reshape(T, d // 128, 128) * s.cpu().numpy()[:, :, None].astype(np.float64)
    np.testing.assert_array_equal(s.cpu().numpy(), scale_ref)
    np.testing.assert_array_equal(deq.reshape(T, d), deq_ref)


@pytest.fixture(scope="module")
def r1_fp8():
    print("drawing R1-shaped fp8 expert weights on the device", flush=True)
    W = make_expert_weights_torch(R1_FP8, seed=0, device=DEV)
    Wt = caee.pack_weights(W, "fp8")
    torch.cuda.synchronize()
    yield W, Wt
    del W, Wt
    torch.cuda.empty_cache()


@pytest.mark.parametrize("T,tokens,rule,tau", [(64, None, "max", 0.05), (64, [5, 60], "sum", 1.2),
                                               (1, None, "max", 0.0)])
def test_r1_fp8_decode(T, tokens, rule, tau, r1_fp8):
    # tokens None: every token of the batch
    W, Wt = r1_fp8
    inp = make_routing_inputs(R1_FP8, seed=3, T=T, zipf_logit_s=1.1, cost_kind="zipf", n_bins=8)
    print(f"fp8 R1 T={T} rule={rule} tau={tau}", flush=True)
    got = gpu_layer(R1_FP8, inp, tau, 8, Wt, DEV, rule=rule)
    get, get_sh = getters_dev(W, "fp8")
    ref = oracle_layer(R1_FP8, inp, tau, 8, get, get_sh, tokens=tokens, rule=rule)
    check_route(got, ref, R1_FP8.E)
    toks = list(range(T)) if tokens is None else tokens
    rel = check_y(got["y"][toks], ref["y"], 6e-2)
    print(f"  {len(toks)} tokens: max|err|/max|ref| = {rel:.3e}", flush=True)


# The last batch of a layer of more than 1 GB whose experts of up to 32 rows are
# small chunks (under 10 rows per expert), and the first whose chunks are all big.
@pytest.mark.parametrize("T", [319, 320])
def test_r1_fp8_all_big_line(T, r1_fp8):
    W, Wt = r1_fp8
    inp = make_routing_inputs(R1_FP8, seed=6, T=T, zipf_logit_s=1.1, n_bins=8)
    print(f"fp8 R1 T={T}", flush=True)
    got = gpu_layer(R1_FP8, inp, 0.0, 8, Wt, DEV)
    tokens = [0, T // 2, T - 1]
    get, get_sh = getters_dev(W, "fp8")
    ref = oracle_layer(R1_FP8, inp, 0.0, 8, get, get_sh, tokens=tokens)
    check_route(got, ref, R1_FP8.E)
    check_y(got["y"][tokens], ref["y"], 6e-2)


def prefill_subset(topk_ids, T, n_shared, n=256, chunk=128, seed=0):
    """A fixed subset of ``n`` tokens of a prefill batch that covers the
    edges of the FFN's work items: an expert slot with r rows is cut into
    ceil(r / chunk) near-equal pieces of consecutive rows (tokens in
    ascending order), so the first and last token of every piece of the
    shared experts (which hold every token) and of every routed expert cut
    into two or three pieces are included; the rest is drawn at random."""
    pick = set()
    def edges(rows):
        r = len(rows)
        pieces = -(-r // chunk)
        size = -(-r // pieces)
        for c in range(pieces):
            pick.add(int(rows[c * size]))
            pick.add(int(rows[min(r, (c + 1) * size) - 1]))
    if n_shared:
        edges(np.arange(T))
    multi = []
    for e in range(int(topk_ids.max()) + 1):
        rows = np.flatnonzero((topk_ids == e).any(axis=1))
        if chunk < len(rows) <= 3 * chunk:
            multi.append((e, rows))
    for e, rows in multi[:24]:
        edges(rows)
    rng = np.random.default_rng(seed)
    rest = [t for t in rng.permutation(T).tolist() if t not in pick]
    out = sorted(pick) + rest[:max(0, n - len(pick))]
    return sorted(out)[:max(n, len(pick))], len(multi)


def test_r1_fp8_prefill(r1_fp8):
    W, Wt = r1_fp8
    T = 4096
    inp = make_routing_inputs(R1_FP8, seed=4, T=T, cost_kind="zipf", n_bins=8)
    print("fp8 R1 prefill T=4096", flush=True)
    got = gpu_layer(R1_FP8, inp, 0.05, 8, Wt, DEV)
    tokens, n_multi = prefill_subset(got["topk_ids"], T, R1_FP8.n_shared)
    assert n_multi >= 2, "the batch has fewer than two experts cut into two or three pieces"
    print(f"  {len(tokens)} tokens ({n_multi} routed experts of two or three pieces)", flush=True)
    get, get_sh = getters_dev(W, "fp8")
    ref = oracle_layer(R1_FP8, inp, 0.05, 8, get, get_sh, tokens=tokens)
    check_route(got, ref, R1_FP8.E)
    rel = check_y(got["y"][tokens], ref["y"], 6e-2)
    print(f"  max|err|/max|ref| = {rel:.3e}", flush=True)
