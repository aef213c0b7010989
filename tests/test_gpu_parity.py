"""GPU parity: the HIP library, called through its C ABI (ctypes binding), against the CPU oracle.

Bars: routing (top-k indices) and bucketing bit-exact; gate weights within 1e-6; outputs within
max|y - y_ref| / max|y_ref| <= 5e-3 (bf16 storage, fp32 accumulation) or 1e-5 (fp32).
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import margin
import paper_2405_13053_amd as m
from gen import inputs as gen
from tests import util

pytestmark = pytest.mark.gpu

LS = gen.LayerShape


def _np(t):
    return t.detach().cpu().numpy()


# ------------------------------------------------------------------------------ gate / routing
GATE_SHAPES = [
    LS(64, 256, 256, 4, 8, 2, 2.0, "f32", "uniform", "cfg1"),
    LS(257, 1024, 64, 28, 8, 2, 2.0, "bf16", "uniform", "ragged-T"),
    LS(1000, 4096, 64, 28, 8, 2, 2.0, "bf16", "zipf", "zipf"),
    LS(130, 520, 64, 37, 8, 3, 2.0, "bf16", "uniform", "N>32,odd-K"),
    LS(96, 5120, 64, 64, 8, 8, 2.0, "bf16", "uniform", "N=64,k=8"),
    LS(33, 264, 64, 5, 8, 1, 2.0, "f32", "zipf", "top1"),
    LS(1, 4096, 64, 28, 8, 2, 2.0, "bf16", "uniform", "T=1"),
]


@pytest.mark.parametrize("shape", GATE_SHAPES, ids=lambda s: s.name)
def test_gate_topk_matches_oracle(shape):
    ops, dev = util.make_case(shape, seed=11)
    g64, g32, idx_ref, w_ref = util.oracle_routing(ops, shape.k)
    idx, w, logits = m.gate_topk(dev["x"], dev["W_gate"], dev["bias"], shape.k, want_logits=True)
    torch.cuda.synchronize()
    idx, w, logits = _np(idx), _np(w), _np(logits)
    # (1) logit accuracy: fp32 accumulation noise, scaled by the sum of |terms|
    mag = np.abs(ops["x"].astype(np.float64)) @ np.abs(ops["W_gate"].astype(np.float64))
    if ops["bias"] is not None:
        mag = mag + np.abs(ops["bias"].astype(np.float64))
    assert np.all(np.abs(logits - g64) <= 8 * 2.0 ** -24 * mag + 1e-30)
    # (2) selection logic on the GPU's own logits: zero tolerance
    idx_self, w_self = oracle.topk_softmax(logits, shape.k)
    assert np.array_equal(idx, idx_self)
    np.testing.assert_allclose(w, w_self, rtol=0, atol=1e-6)
    # (3) routing equals the oracle's, bit-exact (inputs are margin-conditioned)
    assert np.array_equal(idx, idx_ref)
    # (4) Eq. 3 weights vs the oracle's: d(softmax)/d(logit) <= 1/4 per logit, so the logit noise of (1)
    #     moves a weight by at most half the largest logit deviation, on top of the 1e-6 of (2)
    np.testing.assert_allclose(w, w_ref, rtol=0, atol=1e-6 + 0.5 * float(np.abs(logits - g32).max()))
    np.testing.assert_allclose(w.sum(axis=1), 1.0, rtol=0, atol=1e-6)
    assert np.all(w > 0)


def test_gate_selection_logic_on_unconditioned_inputs():
    """Near ties are allowed to resolve either way vs. fp64, but never against the GPU's own logits."""
    shape = LS(3000, 512, 64, 28, 8, 2, 2.0, "bf16")
    ops, dev = util.make_case(shape, seed=5, condition=False)
    idx, w, logits = m.gate_topk(dev["x"], dev["W_gate"], None, 2, want_logits=True)
    idx_self, _ = oracle.topk_softmax(_np(logits), 2)
    assert np.array_equal(_np(idx), idx_self)


def test_gate_exact_ties_lowest_index_first():
    shape = LS(200, 512, 64, 12, 8, 4, 2.0, "bf16")
    ops, dev = util.make_case(shape, seed=6, condition=False)
    Wg = ops["W_gate"].copy()
    Wg[:, 7] = Wg[:, 2]          # identical columns -> bit-identical logits in any summation order
    Wg[:, 9] = Wg[:, 2]
    idx, w, logits = m.gate_topk(dev["x"], util.to_dev(Wg, torch.float32), None, 4, want_logits=True)
    logits = _np(logits)
    assert np.array_equal(logits[:, 2], logits[:, 7]) and np.array_equal(logits[:, 2], logits[:, 9])
    idx_self, _ = oracle.topk_softmax(logits, 4)
    assert np.array_equal(_np(idx), idx_self)
    # all-zero gate with k = N: every logit ties, order is 0..N-1 and w = 1/N
    z = torch.zeros((512, 12), dtype=torch.float32, device="cuda")
    idx, w, _ = m.gate_topk(dev["x"], z, None, 8)
    assert np.array_equal(_np(idx), np.tile(np.arange(8, dtype=np.int32), (200, 1)))
    np.testing.assert_allclose(_np(w), 1.0 / 8, rtol=0, atol=1e-7)


def test_gate_temperature():
    shape = LS(100, 256, 64, 6, 8, 2, 2.0, "f32")
    ops, dev = util.make_case(shape, seed=7)
    idx, w, logits = m.gate_topk(dev["x"], dev["W_gate"], None, 2, inv_temperature=1 / 15.0, want_logits=True)
    idx_ref, w_ref = oracle.topk_softmax(_np(logits), 2, temperature=15.0)
    assert np.array_equal(_np(idx), idx_ref)
    np.testing.assert_allclose(_np(w), w_ref, rtol=0, atol=1e-6)


# ------------------------------------------------------------------------------------ bucketing
@pytest.mark.parametrize("T,k,N,mode", [(64, 2, 4, "uniform"), (4096, 2, 28, "uniform"), (8192, 2, 28, "zipf"),
                                        (1023, 3, 64, "uniform"), (513, 1, 7, "one-bucket"), (1, 2, 28, "uniform"),
                                        (16384, 2, 28, "zipf"), (700, 8, 9, "uniform")])
def test_bucket_tokens_bit_exact(T, k, N, mode):
    rng = np.random.default_rng(T * 131 + k)
    if mode == "one-bucket":
        idx = np.full((T, k), 3, dtype=np.int32)
    else:
        # k distinct adapters per token, drawn with probabilities p (Gumbel top-k)
        p = 1.0 / (np.arange(N) + 1.0) ** 2 if mode == "zipf" else np.ones(N)
        scores = np.log(p)[None, :] + rng.gumbel(size=(T, N))
        idx = np.argsort(-scores, axis=1)[:, :k].astype(np.int32)
    c_ref, o_ref, tok_ref, slot_ref = oracle.bucket(idx, N)
    c, o, tok, slot = m.bucket_tokens(torch.from_numpy(idx).cuda(), N)
    assert np.array_equal(_np(c), c_ref)
    assert np.array_equal(_np(o), o_ref)
    assert np.array_equal(_np(tok), tok_ref)
    assert np.array_equal(_np(slot), slot_ref)
    assert int(_np(c).sum()) == T * k


# ------------------------------------------------------------------------------------ LoRA term
LORA_SHAPES = [
    LS(64, 256, 256, 4, 8, 2, 2.0, "f32", "uniform", "cfg1"),
    LS(300, 512, 1032, 28, 8, 2, 2.0, "bf16", "uniform", "bf16-r8"),
    LS(517, 1024, 520, 28, 16, 2, 2.0, "bf16", "zipf", "bf16-r16-zipf"),
    LS(70, 264, 136, 6, 5, 3, 0.5, "bf16", "uniform", "odd-r"),
    LS(40, 128, 64, 3, 64, 1, 1.0, "f32", "uniform", "r64-top1"),
    # >= 16384 (token, slot) pairs: the shrink runs whole-K tiles and the scatter clears the expand operand
    LS(8300, 520, 136, 28, 16, 2, 2.0, "bf16", "zipf", "whole-K-shrink-ragged"),
    LS(4200, 264, 72, 5, 40, 4, 1.0, "bf16", "uniform", "whole-K-shrink-r40"),
]


@pytest.mark.parametrize("shape", LORA_SHAPES, ids=lambda s: s.name)
def test_lora_forward_matches_oracle(shape):
    ops, dev = util.make_case(shape, seed=21)
    _, _, idx_ref, w_ref = util.oracle_routing(ops, shape.k)
    delta_ref = oracle.lora_delta(ops["x"], ops["A"], ops["B"], idx_ref, w_ref, shape.scale)
    idx_d = torch.from_numpy(idx_ref).cuda()
    w_d = torch.from_numpy(w_ref.astype(np.float32)).cuda()
    out = m.lora_forward(dev["x"], dev["A"], dev["B"], idx_d, w_d, shape.scale)
    assert util.rel_max_err(out, delta_ref) <= util.tol(shape)
    # accumulate=1 on top of the base projection
    base_ref = oracle.base(ops["x"], ops["W"])
    out2 = util.to_dev(base_ref.astype(np.float32), util.torch_dtype(shape))
    base_stored = out2.to(torch.float64).cpu().numpy()
    m.lora_forward(dev["x"], dev["A"], dev["B"], idx_d, w_d, shape.scale, out=out2, accumulate=True)
    assert util.rel_max_err(out2, base_stored + delta_ref) <= util.tol(shape)


# --------------------------------------------------------------------------------- base GEMM
@pytest.mark.parametrize("T,d_in,d_out,dtype", [(64, 256, 256, "f32"), (300, 520, 264, "bf16"),
                                                (1024, 1024, 1024, "bf16"), (17, 4096, 72, "bf16"),
                                                (1300, 192, 4104, "bf16"),      # 256 x 128 tiles, ragged both ways
                                                (2600, 128, 4104, "bf16"),      # 256 x 256 tiles, ragged both ways
                                                (4400, 128, 4104, "bf16")])     # 306 big tiles: 128 x 128 tiles instead
def test_base_gemm_matches_oracle(T, d_in, d_out, dtype):
    shape = LS(T, d_in, d_out, 2, 2, 1, 1.0, dtype)
    ops, dev = util.make_case(shape, seed=31, condition=False)
    out = m.base_gemm(dev["x"], dev["W"])
    assert util.rel_max_err(out, oracle.base(ops["x"], ops["W"])) <= util.tol(shape)


# The 16x16x32 kernel at the edges of its K loop in each of its tile shapes, ragged in both directions: 1, 2 and 3 K tiles; the
# first and the second unrolled trip of six tiles (256x256, entered from 8 and 14 K tiles) and of twelve (192 to 256 rows of
# 128 columns, from 15 and 27) with none, one and more tiles left.
@pytest.mark.parametrize("d_in", [64, 128, 192, 448, 512, 576, 832, 896, 960, 1024, 1088, 1152, 1664, 1728, 1792])
@pytest.mark.parametrize("T,d_out", [(2600, 4104), (1300, 4104), (300, 264), (1100, 4104), (1500, 4104), (1700, 4104), (1700, 5128)],
                         ids=["256x256", "192x128", "128x128", "160x128", "224x128", "256x128", "128x128-two-per-CU"])
def test_base_gemm_k_loop_edges(T, d_out, d_in):
    shape = LS(T, d_in, d_out, 2, 2, 1, 1.0, "bf16")
    _, dev = util.make_case(shape, seed=32, condition=False)
    out = m.base_gemm(dev["x"], dev["W"])
    ref = dev["x"].double() @ dev["W"].double().t().contiguous()
    # one bf16 rounding of an fp32 sum: half an ulp (2^-9 of the value), fp32 summation error far below it
    assert float(((out.double() - ref).abs() - 2.0 ** -8 * ref.abs()).max()) <= 1e-4


# Widths that leave a partial K tile (1 to 7 chunks of 8 columns; up to 32 columns of it are one k-step), alone and behind 1 to
# 28 whole tiles, in each tile shape and at up to 64 tokens.  Where a load ran past d_in it would bring the first columns of the
# next row: one row of x and one of W start with infinities, which may reach that token's and that column's outputs alone.
@pytest.mark.parametrize("d_in", [8, 32, 40, 56, 72, 136, 184, 232, 456, 520, 1000, 1048, 1112, 1800])
@pytest.mark.parametrize("T,d_out", [(2600, 4104), (1300, 4104), (300, 264), (1100, 4104), (1500, 4104), (1700, 4104), (1700, 5128),
                                     (63, 200), (1, 4104)],
                         ids=["256x256", "192x128", "128x128", "160x128", "224x128", "256x128", "128x128-two-per-CU", "64x64", "one"])
def test_base_gemm_partial_k_tile(T, d_out, d_in):
    shape = LS(T, d_in, d_out, 2, 2, 1, 1.0, "bf16")
    _, dev = util.make_case(shape, seed=37, condition=False)
    t, c = T // 2, d_out // 2
    dev["x"][t, :8] = float("inf")
    dev["W"][c, :8] = float("inf")
    out = m.base_gemm(dev["x"], dev["W"]).double()
    ref = dev["x"].double() @ dev["W"].double().t().contiguous()
    assert not torch.isfinite(out[t]).any() and not torch.isfinite(out[:, c]).any()
    out[t], out[:, c], ref[t], ref[:, c] = 0.0, 0.0, 0.0, 0.0
    # one bf16 rounding of an fp32 sum: half an ulp (2^-9 of the value), fp32 summation error far below it
    assert float(((out - ref).abs() - 2.0 ** -8 * ref.abs()).max()) <= 1e-4


# Base projections of few tokens, tiles of 64 columns: each height at its least and largest batch, ragged in both directions, with
# fewer K tiles than the ring is deep, as many, one more, and partial ones; and the next batch, which takes 128 columns.
@pytest.mark.parametrize("d_in", [8, 64, 256, 320, 328, 384, 1000])
@pytest.mark.parametrize("T,d_out", [(1, 8), (16, 16384), (64, 4104), (192, 4104), (193, 4104), (288, 4104), (289, 4104), (384, 4104),
                                     (385, 4104), (1, 16392), (2048, 72)])
def test_base_gemm_of_few_tokens(T, d_out, d_in):
    _, dev = util.make_case(LS(T, d_in, d_out, 2, 2, 1, 1.0, "bf16"), seed=38, condition=False)
    out = m.base_gemm(dev["x"], dev["W"])
    ref = dev["x"].double() @ dev["W"].double().t().contiguous()
    # one bf16 rounding of an fp32 sum: half an ulp (2^-9 of the value), fp32 summation error far below it
    assert float(((out.double() - ref).abs() - 2.0 ** -8 * ref.abs()).max()) <= 1e-4


# accumulate = 1 in each tile shape: the old output is read, added in fp32 and rounded once; ranks whose last
# extension K tile is a half (N*r % 64 <= 32) and a whole one
@pytest.mark.parametrize("N,r", [(28, 8), (7, 8)], ids=["half-tile", "whole-tile"])
@pytest.mark.parametrize("T,d_out", [(2600, 4104), (1300, 4104), (300, 264), (1100, 4104), (1500, 4104), (1700, 4104), (1700, 5128)],
                         ids=["256x256", "192x128", "128x128", "160x128", "224x128", "256x128", "128x128-two-per-CU"])
def test_lora_accumulate_in_each_tile_shape(T, d_out, N, r):
    shape = LS(T, 64, d_out, N, r, 2, 2.0, "bf16")
    ops, dev = util.make_case(shape, seed=33, condition=False)
    idx, w, _ = m.gate_topk(dev["x"], dev["W_gate"], None, 2)
    old = torch.randn((T, d_out), device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)).bfloat16()
    out = m.lora_forward(dev["x"], dev["A"], dev["B"], idx, w, 2.0, out=old.clone(), accumulate=True)
    ref = oracle.lora_delta(ops["x"], ops["A"], ops["B"], _np(idx), _np(w).astype(np.float64), 2.0)
    assert util.rel_max_err(out, old.double().cpu().numpy() + ref) <= util.tol(shape)


# Routing that leaves most of the expand's K tiles (64 columns of N*r) empty: the first or last tile alone, tiles far
# apart, a rank that straddles tiles, and in the second half of the tokens other adapters than in the first.
@pytest.mark.parametrize("N,r,used", [(28, 8, (27,)), (28, 8, (0, 9)), (64, 32, (3, 40, 63)), (9, 24, (2, 5)), (28, 16, (4,))])
def test_lora_with_unused_adapters(N, r, used):
    T, d_out, k = 700, 264, 2
    shape = LS(T, 128, d_out, N, r, k, 2.0, "bf16")
    ops, dev = util.make_case(shape, seed=34, condition=False)
    rng = np.random.default_rng(5)
    first = np.array(used)
    idx = np.stack([first[rng.integers(0, len(first), T)], np.full(T, 1)], 1).astype(np.int32)   # 1 is in no `used`
    idx[T // 2:, 1] = N // 2
    w = rng.uniform(0.2, 0.8, (T, k)).astype(np.float32)
    out = m.lora_forward(dev["x"], dev["A"], dev["B"], torch.from_numpy(idx).cuda(), torch.from_numpy(w).cuda(), 2.0)
    ref = oracle.lora_delta(ops["x"], ops["A"], ops["B"], idx, w.astype(np.float64), 2.0)
    assert util.rel_max_err(out, ref) <= util.tol(shape)


# The fewest K tiles the extension can have, lora_forward being nothing else: a lone half tile (28 adapters of rank 8, all
# tokens on the last; 4 adapters), and none at all for whole row tiles whose tokens name no adapter (ids outside [0, N));
# any integer as an id; token counts that end inside a 16-byte piece of the ids.
@pytest.mark.parametrize("T,N,r,k,pick", [(301, 28, 8, 1, "last"), (99, 4, 8, 2, "any"), (703, 28, 8, 1, "none-first"),
                                          (703, 28, 8, 3, "any-int-first"), (2601, 64, 32, 8, "any-int-first"),
                                          (389, 28, 12, 5, "none-first"), (65, 28, 8, 1, "any")])
@pytest.mark.parametrize("accumulate", [False, True])
def test_lora_with_a_lone_half_tile_or_none(T, N, r, k, pick, accumulate):
    d_in, d_out = 128, 4104 if T > 2000 else 264
    shape = LS(T, d_in, d_out, N, r, k, 2.0, "bf16")
    ops, dev = util.make_case(shape, seed=36, condition=False)
    rng = np.random.default_rng(7)
    idx = np.argsort(rng.random((T, N)), 1)[:, :k].astype(np.int32)
    if pick == "last":
        idx[:] = N - 1
    w = rng.uniform(0.2, 0.8, (T, k)).astype(np.float32)
    old = torch.randn((T, d_out), device="cuda", generator=torch.Generator(device="cuda").manual_seed(5)).bfloat16()
    given, counts = idx.copy(), w.copy()
    nobody = 256 if pick.endswith("first") else 0
    outside = [N, -1, 2**31 - 1] + ([-2**31, 64, 2**26] if pick == "any-int-first" else [])
    given[:nobody] = np.resize(np.array(outside, np.int32), (nobody, k))
    counts[:nobody] = 0
    out = m.lora_forward(dev["x"], dev["A"], dev["B"], torch.from_numpy(given).cuda(), torch.from_numpy(w).cuda(), 2.0,
                         out=old.clone(), accumulate=accumulate)
    ref = oracle.lora_delta(ops["x"], ops["A"], ops["B"], idx, counts.astype(np.float64), 2.0)
    if accumulate:
        ref = ref + old.double().cpu().numpy()
    assert torch.equal(out[:nobody], old[:nobody] if accumulate else torch.zeros_like(old[:nobody]))
    assert util.rel_max_err(out, ref) <= util.tol(shape)


# lora_forward on a given routing on either side of the rule between products of every adapter and bucket lists (T = 64,
# 1024, 4096 tokens; N*r = 256), with ids outside [0, N), accumulate on and off.
@pytest.mark.parametrize("T,d_in,N,r,k", [(64, 128, 28, 8, 2), (65, 128, 28, 8, 2), (1024, 192, 28, 16, 1), (1025, 192, 28, 16, 1),
                                          (4096, 64, 32, 8, 1), (4097, 64, 32, 8, 1), (4097, 64, 32, 8, 2), (300, 320, 3, 24, 3)])
def test_lora_given_routing_on_both_paths(T, d_in, N, r, k):
    d_out = 136
    shape = LS(T, d_in, d_out, N, r, k, 2.0, "bf16")
    ops, dev = util.make_case(shape, seed=35, condition=False)
    rng = np.random.default_rng(6)
    idx = np.argsort(rng.random((T, N)), 1)[:, :k].astype(np.int32)
    w = rng.uniform(0.2, 0.8, (T, k)).astype(np.float32)
    ref = oracle.lora_delta(ops["x"], ops["A"], ops["B"], idx, w.astype(np.float64), 2.0)
    idx_d, w_d = torch.from_numpy(idx).cuda(), torch.from_numpy(w).cuda()
    out = m.lora_forward(dev["x"], dev["A"], dev["B"], idx_d, w_d, 2.0)
    assert util.rel_max_err(out, ref) <= util.tol(shape)
    old = torch.randn((T, d_out), device="cuda", generator=torch.Generator(device="cuda").manual_seed(4)).bfloat16()
    out = m.lora_forward(dev["x"], dev["A"], dev["B"], idx_d, w_d, 2.0, out=old.clone(), accumulate=True)
    assert util.rel_max_err(out, old.double().cpu().numpy() + ref) <= util.tol(shape)
    # ids outside [0, N) count nowhere
    bad = idx_d.clone()
    bad[::7, k - 1] = N
    bad[3::7, k - 1] = -1
    keep = torch.ones_like(w_d)
    keep[::7, k - 1] = 0
    keep[3::7, k - 1] = 0
    out = m.lora_forward(dev["x"], dev["A"], dev["B"], bad, w_d, 2.0)
    ref = oracle.lora_delta(ops["x"], ops["A"], ops["B"], idx, (w_d * keep).cpu().numpy().astype(np.float64), 2.0)
    assert util.rel_max_err(out, ref) <= util.tol(shape)


@pytest.mark.parametrize("T,N,r", [(65, 28, 8), (1025, 28, 16)], ids=["dense", "bucketed"])
def test_lora_adapter_named_twice_counts_in_its_last_slot(T, N, r):
    shape = LS(T, 192, 136, N, r, 3, 2.0, "bf16")
    ops, dev = util.make_case(shape, seed=37, condition=False)
    rng = np.random.default_rng(8)
    idx = np.argsort(rng.random((T, N)), 1)[:, :3].astype(np.int32)
    w = rng.uniform(0.2, 0.8, (T, 3)).astype(np.float32)
    counts = w.copy()
    idx[::2, 2] = idx[::2, 0]
    counts[::2, 0] = 0
    idx[::4, 1] = idx[::4, 0]
    counts[::4, 1] = 0
    out = m.lora_forward(dev["x"], dev["A"], dev["B"], torch.from_numpy(idx).cuda(), torch.from_numpy(w).cuda(), 2.0)
    ref = oracle.lora_delta(ops["x"], ops["A"], ops["B"], idx, counts.astype(np.float64), 2.0)
    assert util.rel_max_err(out, ref) <= util.tol(shape)


# --------------------------------------------------------------------------------- whole layer
LAYER_SHAPES = [
    LS(64, 256, 256, 4, 8, 2, 2.0, "f32", "uniform", "cfg1"),
    LS(333, 512, 776, 28, 8, 2, 2.0, "bf16", "uniform", "bf16-ragged"),
    LS(512, 1024, 512, 28, 16, 2, 2.0, "bf16", "zipf", "bf16-r16-zipf"),
    LS(50, 264, 136, 7, 5, 3, 1.5, "f32", "uniform", "f32-odd"),
    LS(1, 8, 8, 1, 1, 1, 1.0, "f32", "uniform", "f32-smallest"),
    LS(9, 72, 1032, 64, 64, 8, 0.5, "f32", "zipf", "f32-N64-r64-k8"),
    LS(517, 24, 552, 28, 8, 2, 2.0, "f32", "uniform", "f32-32x32-tiles-half-K-step"),
    LS(1537, 40, 2056, 5, 8, 2, 2.0, "f32", "zipf", "f32-128x128-tiles"),
    LS(2049, 72, 2056, 28, 64, 4, 0.5, "f32", "zipf", "f32-expand-apart"),
    LS(7, 40, 1288, 9, 5, 8, 0.5, "f32", "uniform", "f32-expand-apart-r5"),
    LS(100, 512, 256, 28, 8, 1, 2.0, "bf16", "uniform", "top1"),
]


def _check_layer(shape, seed, layer=0, rows="all", inv_temperature=1.0):
    ops, dev = util.make_case(shape, seed, layer)
    g64 = oracle.gate_logits(ops["x"], ops["W_gate"], ops["bias"])
    g32 = g64.astype(np.float32)
    idx_ref, w_ref = oracle.topk_softmax(g32, shape.k, temperature=1.0 / inv_temperature)
    out, idx, w = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], dev["bias"], dev["A"], dev["B"], shape.k,
                                   shape.scale, return_routing=True, inv_temperature=inv_temperature)
    torch.cuda.synchronize()
    assert np.array_equal(_np(idx), idx_ref), "routing differs from the oracle"
    assert np.all(np.abs(_np(w) - w_ref) <= util.weight_bound(ops, idx_ref, inv_temperature)), "gate weights off"
    if rows == "all":
        sel = None
        y_gpu = out
    else:
        c, o, tok, _ = oracle.bucket(idx_ref, shape.N)
        sel = util.sample_rows(shape.T, c, o, tok)
        y_gpu = out[torch.from_numpy(sel.astype(np.int64)).cuda()]
    ref = oracle.linear_forward(ops["x"], ops["W"], ops["W_gate"], ops["bias"], ops["A"], ops["B"], shape.k,
                                shape.scale, rows=sel, temperature=1.0 / inv_temperature)
    err = util.rel_max_err(y_gpu, ref["y"])
    assert err <= util.tol(shape), f"{shape.name}: rel err {err:.3e}"
    # weights packed once (meteora_pack_weights) instead of per call: the same kernels on the same layouts
    packed = m.pack_weights(dev["W_gate"], dev["A"], dev["B"])
    out_p, idx_p, w_p = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], dev["bias"], dev["A"], dev["B"],
                                         shape.k, shape.scale, return_routing=True, packed=packed,
                                         inv_temperature=inv_temperature)
    assert torch.equal(out_p, out) and torch.equal(idx_p, idx) and torch.equal(w_p, w)
    return out


@pytest.mark.parametrize("shape", LAYER_SHAPES, ids=lambda s: s.name)
def test_linear_forward_matches_oracle(shape):
    _check_layer(shape, seed=41)


# adapters in chunks of tokens: 16 up to 2048 tokens, 64 above (33 adapters of a few tiles, and 40 of up to 640 rows of Wcat, without lists)
@pytest.mark.parametrize("T,d_in,N,k", [(65, 136, 64, 8), (95, 4616, 33, 3), (2047, 72, 64, 4), (2048, 136, 40, 1), (2049, 136, 64, 4)])
def test_bucketing_chunk_sizes(T, d_in, N, k):
    _check_layer(LS(T, d_in, 136, N, 8, k, 2.0, "bf16", "zipf", "chunks"), seed=63, rows="sample")


# bucketed sequence (more than 640 rows of Wcat, and more than a few output tiles, too few inputs for two K splits or too many rows of
# B) at the same chunk sizes, and with more than one K slice of 512 inputs
@pytest.mark.parametrize("T,d_in,d_out,N,r,k", [
    (2048, 136, 136, 64, 8, 4), (1600, 4616, 136, 64, 32, 3), (95, 4616, 7048, 64, 64, 8), (30, 4616, 8264, 64, 64, 8)])
def test_bucketed_sequence(T, d_in, d_out, N, r, k):
    _check_layer(LS(T, d_in, d_out, N, r, k, 2.0 if r == 8 else 0.5, "bf16", "zipf", "chunks"), seed=63, rows="sample")


def _sequence(T, d_in, d_out, N, r, k, dtype="bf16"):
    """Which launches a layer call takes, from what they write."""
    regs = {name for name, _, _, written in m.workspace_regions(T, d_in, d_out, N, r, k, dtype, True) if written > 0}
    if dtype == "f32":
        return "fp32"
    return next(name for region, name in (("gpart", "decode"), ("spart", "few-tile"), ("dpart", "dense"), ("partials", "bucketed"))
                if region in regs)


# what the tests of a sequence run, here and below
@pytest.mark.parametrize("sequence,shapes", [
    ("decode", [(48, 1024, 520, 28, 8, 2), (48, 1024, 520, 28, 8, 1), (33, 1024, 520, 28, 8, 2)]),
    ("few-tile", [(200, 1024, 1096, 28, 8, 2), (200, 1024, 1096, 28, 8, 1), (700, 512, 264, 28, 12, 2), (700, 512, 264, 28, 12, 1),
                  (333, 1024, 520, 28, 8, 2), (400, 1024, 520, 28, 16, 2), (95, 4616, 136, 33, 8, 3)]),
    ("dense", [(2500, 512, 2056, 28, 8, 2), (2500, 512, 2056, 28, 8, 1), (2048, 136, 136, 40, 8, 1), (70000, 256, 264, 28, 8, 2)]),
    ("bucketed", [(1300, 320, 2056, 64, 32, 4), (1300, 320, 2056, 64, 32, 1), (65, 136, 136, 64, 8, 8), (2047, 72, 136, 64, 8, 4),
                  (2048, 136, 136, 64, 8, 4), (2049, 136, 136, 64, 8, 4), (1600, 4616, 136, 64, 32, 3), (95, 4616, 7048, 64, 64, 8),
                  (30, 4616, 8264, 64, 64, 8), (70000, 256, 264, 28, 12, 2)])])
def test_each_shape_takes_its_sequence(sequence, shapes):
    assert [_sequence(*s) for s in shapes] == [sequence] * len(shapes)


# fp32 layers with few adapters in one launch: tiles of 16 tokens and 16 columns, K in steps of 16 over four wavefronts
@pytest.mark.parametrize("T,d_in,d_out,N,r,k", [
    (1, 8, 8, 1, 1, 1), (16, 16, 16, 16, 2, 8), (17, 24, 24, 16, 4, 3), (33, 72, 264, 4, 8, 2), (15, 512, 8, 4, 8, 1),
    (64, 328, 136, 2, 16, 2), (129, 64, 904, 7, 8, 3), (40, 168, 40, 1, 64, 1), (9, 136, 4096, 5, 12, 4),
    (16, 16, 16, 16, 2, 3), (40, 168, 40, 1, 32, 1), (77, 128, 136, 13, 4, 4)])
def test_fp32_layer_in_one_launch(T, d_in, d_out, N, r, k):
    _check_layer(LS(T, d_in, d_out, N, r, k, 2.0, "f32", "zipf", "f32-one-launch"), seed=62)


# two workgroups per CU, and at most one, have a kernel each
@pytest.mark.parametrize("T,d_in,d_out,N,r,k", [(129, 40, 520, 4, 8, 2), (512, 256, 256, 4, 8, 2), (256, 248, 256, 4, 8, 4)])
def test_fp32_layer_in_one_launch_around_one_workgroup_per_cu(T, d_in, d_out, N, r, k):
    _check_layer(LS(T, d_in, d_out, N, r, k, 2.0, "f32", "uniform", "f32-two-per-CU"), seed=71)


# fp32 routing is one sum in one order, whichever launches run: gate_topk, the layer in one launch, the layer in two or three
@pytest.mark.parametrize("d_in,d_out,N,r,k", [
    (256, 256, 4, 8, 2), (8, 8, 1, 1, 1), (256, 256, 16, 2, 8), (72, 264, 16, 4, 3), (512, 8, 4, 8, 1), (328, 136, 2, 16, 2),
    (64, 904, 7, 8, 3), (168, 40, 1, 64, 1), (248, 40, 11, 2, 4), (200, 64, 3, 8, 3), (128, 256, 16, 2, 2), (256, 264, 1, 32, 1),
    (160, 72, 5, 8, 4), (120, 72, 9, 3, 4)])
def test_fp32_routing_does_not_depend_on_the_launches(d_in, d_out, N, r, k):
    shape = LS(4096, d_in, d_out, N, r, k, 2.0, "f32", "zipf", "f32-routing")
    _, dev = util.make_case(shape, seed=66, condition=False)
    idx_ref, w_ref, _ = m.gate_topk(dev["x"], dev["W_gate"], dev["bias"], k)
    for T in (1, 5, 16, 64, 129, 4096):   # 4096 tokens never run in one launch for these widths, except the narrowest
        _, idx, w = m.linear_forward(dev["x"][:T], dev["W"], dev["W_gate"], dev["bias"], dev["A"], dev["B"], k, 2.0,
                                     return_routing=True)
        torch.cuda.synchronize()
        assert torch.equal(idx, idx_ref[:T]), f"T = {T}: adapters differ"
        assert torch.equal(w, w_ref[:T]), f"T = {T}: weights differ"


# row tiles of 128 outputs and of 320 (r = 8), 544 (16) or 320 (7 adapters of 32) rows of Wcat share 256 CUs; up to 8 splits a
# round of the tail, above 16 never (S: splits for the three adapter sets)
@pytest.mark.parametrize("d_in,d_out,S", [
    (512, 24584, (1, 1, 1)), (512, 13832, (2, 2, 2)), (768, 9224, (3, 3, 3)), (1280, 5640, (5, 5, 5)), (4096, 264, (8, 8, 8)),
    (8384, 264, (16, 16, 16)), (8384, 2056, (12, 11, 12)), (6464, 2056, (12, 8, 12)), (6464, 1416, (8, 15, 8))])
@pytest.mark.parametrize("adapters", range(3), ids=["r8", "r16", "r32"])
def test_decode_tail_at_each_split_count(d_in, d_out, S, adapters):
    N, r, k = [(28, 8, 2), (28, 16, 1), (7, 32, 3)][adapters]
    regs = {name: written for name, _, _, written in m.workspace_regions(5, d_in, d_out, N, r, k, "bf16", True)}
    assert regs["splitk"] == S[adapters] * 5 * d_out * 4
    _check_layer(LS(5, d_in, d_out, N, r, k, 2.0, "bf16", "zipf", "tail"), seed=61)


@pytest.mark.parametrize("d_in,same_kernel", [(128, True), (512, False)])
def test_linear_forward_zero_B_is_base_and_deterministic(d_in, same_kernel):
    """B = 0: the layer is the base projection.  d_in = 128: the same GEMM kernel as meteora_base_gemm runs, equal
    bits; d_in = 512: this batch's projection is split along K (other fp32 summation order than the one-sweep
    base GEMM), so the bf16 results agree up to the rounding of sums that differ in their last bits."""
    shape = LS(200, d_in, 520, 28, 8, 2, 2.0, "bf16")
    ops, dev = util.make_case(shape, seed=42)
    zB = torch.zeros_like(dev["B"])
    y0 = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], None, dev["A"], zB, 2, 2.0)
    yb = m.base_gemm(dev["x"], dev["W"])
    if same_kernel:
        assert torch.equal(y0, yb)
    else:
        diff = (y0.float() - yb.float()).abs()
        assert float((diff / yb.float().abs().clamp_min(1e-3)).max()) <= 2.0 ** -7      # one bf16 ulp
        assert float((diff > 0).float().mean()) <= 0.02
    y1 = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], None, dev["A"], dev["B"], 2, 2.0)
    y2 = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], None, dev["A"], dev["B"], 2, 2.0)
    assert torch.equal(y1, y2)


def test_packed_weights_serve_many_batches():
    """One blob, two different batches and batch sizes: each equals the per-call-packing result."""
    shape = LS(333, 1024, 776, 28, 8, 2, 2.0, "bf16")
    ops, dev = util.make_case(shape, seed=44)
    packed = m.pack_weights(dev["W_gate"], dev["A"], dev["B"])
    assert packed.numel() == m.packed_bytes(1024, 776, 28, 8, "bf16")
    for rows in (slice(0, 333), slice(17, 150)):
        x = dev["x"][rows].contiguous()
        y_ref = m.linear_forward(x, dev["W"], dev["W_gate"], None, dev["A"], dev["B"], 2, 2.0)
        y = m.linear_forward(x, dev["W"], dev["W_gate"], None, dev["A"], dev["B"], 2, 2.0, packed=packed)
        assert torch.equal(y, y_ref)


SMALL_BATCH_SHAPES = [
    LS(1, 512, 256, 28, 8, 2, 2.0, "bf16", "uniform", "T=1"),
    LS(64, 1024, 776, 12, 16, 3, 1.5, "bf16", "zipf", "T=64-r16-k3-bias-two-launch"),
    LS(40, 4096, 1032, 28, 8, 2, 2.0, "bf16", "uniform", "T=40-ragged-tiles"),
    LS(7, 264, 136, 5, 16, 1, 1.0, "bf16", "zipf", "T=7-r16-top1-ragged"),
    LS(64, 1024, 520, 64, 32, 8, 0.5, "bf16", "uniform", "T=64-N64-r32-k8"),
    LS(33, 5120, 264, 28, 8, 2, 2.0, "bf16", "zipf", "T=33-decode-shape"),
    LS(48, 1024, 520, 28, 16, 2, 2.0, "bf16", "uniform", "T=48-r16-N28-two-launch"),
    # the decode tail's loops: k*r = 256 shrink values per token (four groups of 64 / r slots), a row of 513
    # 8-column pieces (nine stretches, the last with one active lane), top-1
    LS(50, 1024, 776, 16, 32, 8, 0.5, "bf16", "zipf", "T=50-N16-r32-k8-tail"),
    LS(9, 1024, 4104, 28, 8, 8, 1.0, "bf16", "uniform", "T=9-k8-ragged-stretch"),
    LS(64, 2048, 1544, 28, 8, 1, 2.0, "bf16", "zipf", "T=64-top1-tail"),
    # the launch that streams W: a half-empty last K step, token blocks of 16 at their edges, a ragged row tile
    LS(16, 576, 264, 28, 8, 2, 2.0, "bf16", "uniform", "T=16-half-K-step"),
    LS(17, 1088, 136, 28, 16, 2, 2.0, "bf16", "zipf", "T=17-half-K-step"),
    LS(32, 1600, 1288, 28, 8, 2, 2.0, "bf16", "uniform", "T=32-half-K-step"),
    # 131 and 89 row tiles: runs that cut row tiles at any K step; 258: runs that are longer than a row tile
    LS(33, 512, 16384, 28, 8, 2, 2.0, "bf16", "uniform", "T=33-runs"),
    LS(17, 576, 11008, 28, 8, 2, 2.0, "bf16", "uniform", "T=17-89-row-tiles-runs"),
    LS(5, 512, 32640, 28, 8, 2, 2.0, "bf16", "zipf", "T=5-long-runs"),
]


@pytest.mark.parametrize("shape", SMALL_BATCH_SHAPES, ids=lambda s: s.name)
def test_small_batch_path_matches_oracle_and_gate_entry_point(shape):
    """T <= 64: top-k and shrink run token-major in one launch; same adapters as meteora_gate_topk picks."""
    out = _check_layer(shape, seed=45)
    ops, dev = util.make_case(shape, seed=45)
    _, idx, w = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], dev["bias"], dev["A"], dev["B"], shape.k,
                                 shape.scale, return_routing=True)
    idx_g, w_g, _ = m.gate_topk(dev["x"], dev["W_gate"], dev["bias"], shape.k)
    assert torch.equal(idx, idx_g)
    # where the logits come out of the GEMM's own launch they are summed in another order than the gate kernel's
    assert float((w - w_g).abs().max()) <= 1e-5
    # and the LoRA term alone through the bucketed path gives the same layer output to bf16 accuracy
    base = m.base_gemm(dev["x"], dev["W"])
    full = m.lora_forward(dev["x"], dev["A"], dev["B"], idx, w, shape.scale, out=base.clone(), accumulate=True)
    assert util.rel_max_err(full, out.to(torch.float64).cpu().numpy()) <= 2 * util.tol(shape)


# mid-sized batches (64 < T <= 8192, bf16, r % 8 == 0, d_in % 64 == 0, 96 + N*r <= 320): gate logits and the shrink
# of every adapter in one MFMA launch, selection afterwards; 128x128 tiles up to 4096 tokens, 128x320 above
DENSE_ROUTE_SHAPES = [
    LS(65, 64, 72, 3, 8, 1, 2.0, "bf16", "uniform", "T=65-one-K-tile"),
    LS(129, 320, 264, 9, 24, 4, 0.7, "bf16", "zipf", "T=129-r24-k4-bias"),
    LS(1000, 1088, 520, 28, 8, 2, 2.0, "bf16", "zipf", "T=1000-ragged-K17"),
    LS(700, 512, 256, 7, 32, 7, 1.0, "bf16", "uniform", "T=700-r32-k=N"),
    LS(4097, 256, 136, 28, 8, 2, 2.0, "bf16", "uniform", "T=4097-wide-tiles"),
    LS(5000, 832, 264, 14, 16, 3, 2.0, "bf16", "zipf", "T=5000-r16-wide-tiles"),
    LS(260, 384, 136, 28, 8, 8, 1.0, "bf16", "uniform", "T=260-k8"),
    # few output tiles: the base projection is split along K and the expand runs inside the reduction
    LS(256, 4096, 4096, 28, 8, 2, 2.0, "bf16", "uniform", "T=256-split-K-projection"),
    LS(200, 1024, 1096, 28, 8, 2, 2.0, "bf16", "zipf", "T=200-split-K-ragged-columns"),
    LS(513, 2048, 520, 7, 32, 3, 0.5, "bf16", "uniform", "T=513-split-K-r32"),
    # every height of the split tiles (96 to 256 rows in steps of 32), ragged, few K tiles per split
    LS(66, 512, 1032, 28, 8, 2, 2.0, "bf16", "uniform", "T=66-96-rows"),
    LS(128, 1088, 520, 28, 8, 2, 2.0, "bf16", "zipf", "T=128-128-rows"),
    LS(289, 1024, 1032, 28, 8, 2, 2.0, "bf16", "uniform", "T=289-160-rows"),
    LS(161, 576, 264, 28, 8, 2, 2.0, "bf16", "uniform", "T=161-192-rows"),
    LS(577, 1024, 264, 28, 8, 2, 2.0, "bf16", "uniform", "T=577-224-rows"),
    # so many columns that two workgroups share a CU, tiles of 96 and 128 rows
    LS(67, 768, 16392, 28, 8, 2, 2.0, "bf16", "uniform", "T=67-two-per-CU"),
    LS(128, 832, 17416, 28, 16, 2, 2.0, "bf16", "zipf", "T=128-two-per-CU"),
    # the split projection has more K splits (8) than the routing products alone would take (5)
    LS(3000, 4096, 256, 28, 8, 2, 2.0, "bf16", "uniform", "T=3000-narrow-output-more-splits"),
    # 28 adapters of rank 16: 544 rows of Wcat, several column tiles of the routing products
    LS(70, 512, 264, 28, 16, 2, 2.0, "bf16", "zipf", "T=70-r16-N28-split-K"),
    LS(1000, 1088, 520, 28, 16, 2, 2.0, "bf16", "uniform", "T=1000-r16-N28"),
    LS(4500, 256, 136, 28, 16, 3, 2.0, "bf16", "zipf", "T=4500-r16-N28-two-wide-tiles"),
    LS(300, 320, 200, 32, 16, 4, 1.0, "bf16", "uniform", "T=300-r16-N32-608-rows"),
]


@pytest.mark.parametrize("shape", DENSE_ROUTE_SHAPES, ids=lambda s: s.name)
def test_dense_route_path_matches_oracle_and_bucketed_path(shape):
    """Same routing as meteora_gate_topk bit for bit; the layer equals base GEMM + bucketed LoRA to bf16 accuracy."""
    rows = "all" if shape.T <= 1000 else "sample"
    out = _check_layer(shape, seed=46, rows=rows)
    ops, dev = util.make_case(shape, seed=46)
    _, idx, w = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], dev["bias"], dev["A"], dev["B"], shape.k,
                                 shape.scale, return_routing=True)
    idx_g, w_g, _ = m.gate_topk(dev["x"], dev["W_gate"], dev["bias"], shape.k)
    assert torch.equal(idx, idx_g)
    assert float((w - w_g).abs().max()) <= 1e-5     # the two paths add the logit terms in different orders
    base = m.base_gemm(dev["x"], dev["W"])
    full = m.lora_forward(dev["x"], dev["A"], dev["B"], idx, w, shape.scale, out=base.clone(), accumulate=True)
    assert util.rel_max_err(full, out.to(torch.float64).cpu().numpy()) <= 2 * util.tol(shape)


# Widths that are no multiple of 64 (nor of 128, the decode launch's K step) on every launch sequence: inputs of one chunk, layers
# with fewer K tiles than splits, a partial tile in a split of its own, outputs beyond 256 row tiles, each height of the few-tile form's
# tiles (96 to 256 rows in steps of 32; 96 and 128 also with two workgroups per CU).
@pytest.mark.parametrize("T,d_in,d_out,N,r,k", [
    (1, 8, 8, 28, 8, 2), (64, 24, 136, 28, 16, 1), (49, 320, 2920, 28, 16, 1), (17, 824, 1848, 7, 32, 3), (5, 72, 33000, 28, 8, 2),
    (65, 8, 136, 28, 8, 2), (300, 1000, 264, 28, 8, 2), (130, 1032, 136, 28, 16, 2), (200, 4616, 520, 28, 8, 8), (97, 776, 16392, 28, 8, 2),
    (80, 776, 16392, 28, 8, 2), (66, 1032, 264, 28, 8, 2), (110, 1032, 264, 28, 16, 2), (180, 584, 264, 28, 8, 2), (450, 1096, 520, 28, 8, 2),
    (1100, 1048, 4104, 12, 16, 3), (2500, 136, 2056, 28, 8, 2), (4500, 264, 136, 28, 16, 3), (9000, 72, 264, 28, 8, 1)])
def test_layer_of_any_width(T, d_in, d_out, N, r, k):
    _check_layer(LS(T, d_in, d_out, N, r, k, 2.0, "bf16", "zipf", "any-width"), seed=64, rows="all" if T <= 300 else "sample")


# More than 32 adapters and ranks that are no multiple of 8 or no power of two on every launch sequence: decode with 1 to 16
# splits (equal ones, and runs that cut the gate rows' two tiles in different places), a few hundred tokens, dense routing,
# bucketed.  (Rank 1 with all three adapters: the expand operand and the output are rounded to bf16, 2^-9 each; with rank 1 and
# one adapter a single rounded factor of up to 28 meets sampled outputs of up to 20, 3.98e-3 * 28 / 20 = 5.6e-3 of the largest.)
@pytest.mark.parametrize("N,r,k", [(64, 32, 8), (33, 8, 2), (28, 12, 2), (5, 5, 3), (64, 64, 4), (40, 20, 3), (3, 1, 3), (28, 24, 2)])
@pytest.mark.parametrize("T,d_in,d_out", [(1, 136, 8), (3, 4096, 264), (64, 1024, 776), (17, 512, 11008), (5, 8384, 136),
                                          (65, 512, 264), (130, 1032, 16392), (300, 512, 2056), (1300, 320, 2056)])
def test_layer_with_any_adapters(N, r, k, T, d_in, d_out):
    _check_layer(LS(T, d_in, d_out, N, r, k, 2.0, "bf16", "zipf", "any-adapters"), seed=66, rows="all" if T <= 17 else "sample")


# So many rows of B per token that the dense operand and MFMAs are cheaper than the tail: decode-sized, a few hundred tokens, a group
# with one such member.
@pytest.mark.parametrize("T,d_in,d_out", [(64, 128, 8200), (300, 512, 2056)])
def test_layer_with_many_ranks_per_token(T, d_in, d_out):
    shape = LS(T, d_in, d_out, 64, 64, 8, 0.5, "bf16", "uniform", "many-ranks")
    _check_layer(shape, seed=68, rows="sample")
    shapes, all_ops, members, x, rows = _group_case(T, d_in, (d_out, 136), 64, 64, 8, "uniform", seed=69)
    for mb in members:
        mb["packed"] = m.pack_weights(mb["W_gate"], mb["A"], mb["B"])
    for mb, out in zip(members, m.linear_forward_group(x, members, 8, 0.5)):
        alone = m.linear_forward(x, mb["W"], mb["W_gate"], mb["gate_bias"], mb["A"], mb["B"], 8, 0.5, packed=mb["packed"])
        assert util.rel_max_err(out[rows], alone[rows].to(torch.float64).cpu().numpy()) <= 2 * util.tol(shape)


@pytest.mark.parametrize("T", [9, 200])
def test_padding_of_a_rank_reads_no_other_adapter(T):
    """28 adapters of rank 12, infinities in every adapter but two: tokens that chose only those two see none of them.  (Decode
    and the few-tile form; the fused GEMM multiplies every adapter of a used K tile.)"""
    shape = LS(T, 1024, 264, 28, 12, 2, 2.0, "bf16")
    ops, dev = util.make_case(shape, seed=67, condition=False)
    bias = torch.full((28,), -1e4, device="cuda")
    bias[7] = bias[20] = 0.0
    clean = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], bias, dev["A"], dev["B"], 2, 2.0)
    others = torch.ones(28, dtype=torch.bool, device="cuda")
    others[7] = others[20] = False
    dev["B"][others] = float("inf")
    dev["A"][others] = 0.0     # their shrink is finite: the dense products are of every adapter
    out, idx, _ = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], bias, dev["A"], dev["B"], 2, 2.0, return_routing=True)
    assert sorted(set(_np(idx).ravel().tolist())) == [7, 20]
    assert torch.equal(out, clean)


@pytest.mark.parametrize("d_in,N,r", [(520, 28, 8), (512, 28, 12), (512, 64, 8)], ids=["width", "rank", "adapters"])
def test_a_blob_packed_without_the_routing_rows_is_still_taken(d_in, N, r):
    """Blobs that once ended in front of Wcat: a call that reads it packs it itself, the same bits."""
    for T in (30, 300):
        shape = LS(T, d_in, 264, N, r, 2, 2.0, "bf16")
        _, dev = util.make_case(shape, seed=65)
        whole = m.pack_weights(dev["W_gate"], dev["A"], dev["B"])
        short = whole[:-(3 * (32 if N <= 32 else 64) + N * ((r + 7) // 8 * 8)) * d_in * 2].clone()
        args = (dev["x"], dev["W"], dev["W_gate"], None, dev["A"], dev["B"], 2, 2.0)
        assert torch.equal(m.linear_forward(*args, packed=short), m.linear_forward(*args, packed=whole))
        members = [{"W": dev["W"], "W_gate": dev["W_gate"], "gate_bias": None, "A": dev["A"], "B": dev["B"], "packed": p}
                   for p in (whole, short)]
        one, two = m.linear_forward_group(dev["x"], members, 2, 2.0)
        assert torch.equal(one, two)
        with pytest.raises(m.MeteoraError):
            m.linear_forward(*args, packed=short[:-256].clone())


def test_what_a_blob_without_the_routing_rows_holds_is_not_packed_again():
    """64 adapters of rank 32: a call of many tokens reads the other operands alone and writes none of them into its workspace; a
    few tokens take Wcat from there, and nothing else."""
    bf, (d_in, d_out, N, r, k) = torch.bfloat16, (320, 2056, 64, 32, 4)
    for T, packs in ((1300, ()), (30, ("apack",))):
        shape = LS(T, d_in, d_out, N, r, k, 2.0, "bf16")
        _, dev = util.make_case(shape, seed=72, condition=False)
        whole = m.pack_weights(dev["W_gate"], dev["A"], dev["B"])
        short = whole[:-(3 * 64 + N * r) * d_in * 2].clone()
        ws = torch.full((m.workspace_bytes(T, d_in, d_out, N, r, k, bf),), 0xa5, dtype=torch.uint8, device="cuda")
        args = (dev["x"], dev["W"], dev["W_gate"], None, dev["A"], dev["B"], k, 2.0)
        assert torch.equal(m.linear_forward(*args, packed=short, ws=ws), m.linear_forward(*args, packed=whole))
        regs = {n: (o, s) for n, o, s, _ in m.workspace_regions(T, d_in, d_out, N, r, k, bf, True)}
        for name in ("wsplit", "apack", "btrans"):
            o, s = regs[name]
            assert bool((ws[o:o + s] != 0xa5).any()) == (name in packs), name


# The routing products in each of their tile widths: 128 x 160 (320, 288 and 544 rows of Wcat, one of the last tile's columns ragged)
# with 8, 4 and 2 splits, and beside it with too few inputs for that; 192 to 320 columns for many tokens; partial K tiles.
@pytest.mark.parametrize("T,d_in,d_out,N,r,k", [
    (1100, 2056, 2056, 28, 8, 2), (4000, 1024, 776, 28, 8, 2), (3000, 1096, 1032, 12, 16, 3), (2500, 1032, 1032, 28, 16, 2),
    (4100, 512, 520, 28, 8, 2), (4000, 512, 776, 28, 8, 2), (2300, 1032, 776, 16, 8, 2), (4500, 264, 136, 12, 8, 2),
    (4500, 264, 136, 16, 8, 2), (4500, 264, 136, 20, 8, 1), (4500, 264, 136, 28, 16, 2), (8400, 136, 264, 28, 8, 2), (8400, 136, 264, 30, 16, 8)])
def test_routing_products_in_each_tile_width(T, d_in, d_out, N, r, k):
    _check_layer(LS(T, d_in, d_out, N, r, k, 2.0, "bf16", "zipf", "products"), seed=70, rows="sample")


def test_dense_route_exact_ties_and_zero_gate():
    """Duplicated gate columns tie exactly: the lower index wins on this path too; a zero gate picks 0..k-1."""
    shape = LS(300, 512, 264, 12, 8, 3, 2.0, "bf16")
    ops, dev = util.make_case(shape, seed=47, condition=False)
    Wg = ops["W_gate"].copy()
    Wg[:, 5] = Wg[:, 2]
    Wg[:, 9] = Wg[:, 2]
    for gate in (Wg, np.zeros_like(Wg)):
        g = torch.from_numpy(gate).cuda()
        _, idx, w = m.linear_forward(dev["x"], dev["W"], g, None, dev["A"], dev["B"], 3, 2.0, return_routing=True)
        idx = _np(idx)
        if not gate.any():
            assert np.array_equal(idx, np.tile(np.arange(3, dtype=np.int32), (300, 1)))
            np.testing.assert_allclose(_np(w), 1.0 / 3, rtol=0, atol=1e-7)
        else:
            has2 = (idx == 2).any(axis=1)
            # whenever one of the tied columns is chosen, the lowest of them (2) is among the choices
            assert np.all(has2 | ~((idx == 5) | (idx == 9)).any(axis=1))
            assert np.all(~(idx == 9).any(axis=1) | (idx == 5).any(axis=1))


# A bias of -inf masks an adapter; a token whose input is NaN must not disturb the others.  One shape per place that ranks:
# decode, a few hundred tokens, dense routing, more than 32 adapters, fp32 in two launches, three and one.
@pytest.mark.parametrize("T,d_in,d_out,N,k,dtype", [(33, 512, 136, 28, 3, "bf16"), (200, 512, 264, 28, 3, "bf16"), (2500, 256, 2056, 28, 3, "bf16"),
                                                    (300, 256, 136, 64, 8, "bf16"), (40, 256, 136, 64, 3, "f32"), (40, 256, 1288, 12, 8, "f32"),
                                                    (40, 256, 136, 4, 3, "f32"), (40, 128, 136, 8, 3, "f32")])
def test_masked_adapters_and_a_token_of_nan(T, d_in, d_out, N, k, dtype):
    shape = LS(T, d_in, d_out, N, 8, k, 2.0, dtype)
    ops, dev = util.make_case(shape, seed=57, condition=False)
    bias = np.zeros(N, np.float32)
    open_ = np.array([1, N // 2, N - 1][:max(1, k - 1)])     # fewer than k adapters are left
    bias[np.setdiff1d(np.arange(N), open_)] = -np.inf
    masked = np.setdiff1d(np.arange(N), open_)
    bias_d = torch.from_numpy(bias).cuda()
    x = dev["x"].clone()
    x[T // 2] = float("nan")
    good = torch.arange(T, device="cuda") != T // 2
    for xin in (dev["x"], x):
        rows = good if xin is x else torch.ones_like(good)
        idx_g, w_g, _ = m.gate_topk(xin, dev["W_gate"], bias_d, k)
        out, idx, w = m.linear_forward(xin, dev["W"], dev["W_gate"], bias_d, dev["A"], dev["B"], k, 2.0, return_routing=True)
        for i, wt in ((idx_g, w_g), (idx, w)):
            i, wt = _np(i[rows]), _np(wt[rows])
            assert np.array_equal(np.sort(i[:, :len(open_)], 1), np.tile(open_, (len(i), 1)))
            # the rest are ties at -inf: the lowest of the masked ones, with no weight
            assert np.array_equal(i[:, len(open_):], np.tile(masked[:k - len(open_)], (len(i), 1)))
            assert np.all(wt[:, len(open_):] == 0)
            np.testing.assert_allclose(wt.sum(1), 1, rtol=0, atol=1e-6)
        if xin is x:
            assert torch.equal(out[rows], clean[rows])
            i = _np(idx)
            assert i.min() >= 0 and i.max() < N and all(len(set(r)) == k for r in i)
            assert bool(torch.isnan(out[T // 2]).all())
        clean = out


GRAPH_SHAPES = [
    LS(33, 1024, 520, 28, 8, 2, 2.0, "bf16", "uniform", "graph-decode"),
    LS(333, 1024, 520, 28, 8, 2, 2.0, "bf16", "zipf", "graph-dense-route"),
    LS(400, 1024, 520, 28, 16, 2, 2.0, "bf16", "uniform", "graph-bucketed"),
    # dense routing in front of the fused GEMM (too many output tiles for the split-K form)
    LS(2500, 512, 2056, 28, 8, 2, 2.0, "bf16", "uniform", "graph-dense-route-fused-gemm"),
    # the bucketed sequence (the two of 333 and 400 tokens are of the few-tile form)
    LS(1300, 320, 2056, 64, 32, 4, 0.5, "bf16", "zipf", "graph-lists"),
    LS(64, 256, 256, 4, 8, 2, 2.0, "f32", "uniform", "graph-fp32-one-launch"),
]


@pytest.mark.parametrize("shape", GRAPH_SHAPES, ids=lambda s: s.name)
def test_layer_call_replays_from_a_hip_graph(shape):
    """The library allocates nothing and records no memset: a captured call replays bit-identically on new inputs."""
    ops, dev = util.make_case(shape, seed=48, condition=False)
    dt = util.torch_dtype(shape)
    packed = m.pack_weights(dev["W_gate"], dev["A"], dev["B"])
    ws = torch.empty(m.workspace_bytes(shape.T, shape.d_in, shape.d_out, shape.N, shape.r, shape.k, dt),
                     dtype=torch.uint8, device="cuda")
    x_in = dev["x"].clone()
    out = torch.empty((shape.T, shape.d_out), dtype=dt, device="cuda")
    args = (dev["W"], dev["W_gate"], dev["bias"], dev["A"], dev["B"], shape.k, shape.scale)
    m.linear_forward(x_in, *args, out=out, ws=ws, packed=packed)   # first call sets the kernels' LDS attributes
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            m.linear_forward(x_in, *args, out=out, ws=ws, packed=packed)
    torch.cuda.synchronize()
    gen_t = torch.Generator(device="cuda").manual_seed(5)
    for rep in range(3):
        x_new = torch.randn(dev["x"].shape, generator=gen_t, device="cuda", dtype=torch.float32).to(dt)
        ref = m.linear_forward(x_new, *args, packed=packed)           # eager, own output and workspace
        torch.cuda.synchronize()
        x_in.copy_(x_new)
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref), f"replay {rep} differs from the eager call"


@pytest.mark.parametrize("T", [40, 300, 2500, 9000])
def test_layer_call_does_not_depend_on_workspace_contents(T):
    """The workspace arrives uninitialised: whatever it holds (zeros, all ones, random bytes, the leftovers of other
    calls), the result is the same, call after call."""
    shape = LS(T, 512, 2056, 28, 8, 2, 2.0, "bf16", "zipf", "workspace-garbage")
    ops, dev = util.make_case(shape, seed=55, condition=False)
    dt = torch.bfloat16
    packed = m.pack_weights(dev["W_gate"], dev["A"], dev["B"])
    args = (dev["x"], dev["W"], dev["W_gate"], dev["bias"], dev["A"], dev["B"], shape.k, shape.scale)
    ref, idx_ref, w_ref = m.linear_forward(*args, packed=packed, return_routing=True)
    nbytes = m.workspace_bytes(shape.T, shape.d_in, shape.d_out, shape.N, shape.r, shape.k, dt)
    gen_t = torch.Generator(device="cuda").manual_seed(9)
    fills = [lambda n: torch.zeros(n, dtype=torch.uint8, device="cuda"),
             lambda n: torch.full((n,), 255, dtype=torch.uint8, device="cuda"),
             lambda n: torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda", generator=gen_t),
             lambda n: torch.full((n,), 1, dtype=torch.uint8, device="cuda")]
    for fill in fills:
        ws = fill(nbytes)
        for rep in range(2):   # the second call finds what the first one left
            out, idx, w = m.linear_forward(*args, packed=packed, ws=ws, return_routing=True)
            torch.cuda.synchronize()
            assert torch.equal(idx, idx_ref) and torch.equal(w, w_ref) and torch.equal(out, ref)


@pytest.mark.parametrize("r,N,path", [(12, 28, "bucketed"), (8, 28, "dense"), (16, 28, "rank16")],
                         ids=["bucketed-r12", "dense-r8", "r16"])
def test_many_tokens_small_layer_sampled_rows(r, N, path):
    """T = 70000: index arithmetic at scale on the sequences a large batch can take.  Rank 12 goes through the
    bucketed path (1094 bucketing chunks, whole-K shrink), rank 8 through the dense routing products (320 rows of
    Wcat: every batch size), rank 16 through whichever of the two the tile count of the products selects."""
    shape = LS(70000, 256, 264, N, r, 2, 2.0, "bf16", "zipf", f"T=70000-{path}")
    _check_layer(shape, seed=49, rows="sample")


# ------------------------------------------------------------------ layers that share x (q/k/v, gate/up)
def _group_case(T, d_in, d_outs, N, r, k, routing, seed):
    shapes = [LS(T, d_in, d, N, r, k, 2.0, "bf16", routing, f"member{g}") for g, d in enumerate(d_outs)]
    ops0, dev0 = util.make_case(shapes[0], seed, 0)
    members, all_ops = [], []
    for g, sh in enumerate(shapes):
        ops = gen.make_layer(sh, seed, g)
        ops["x"] = ops0["x"]                      # the members share the (margin-conditioned) input of member 0
        dev = {n: util.to_dev(ops[n], torch.bfloat16) for n in ("W", "A", "B")}
        dev["W_gate"] = util.to_dev(ops["W_gate"], torch.float32)
        dev["gate_bias"] = util.to_dev(ops["bias"], torch.float32)
        all_ops.append(ops)
        members.append(dev)
    # conditioning was done for member 0's gate only: drop the rows that are near-tied for any other member
    keep = np.ones(T, dtype=bool)
    for ops in all_ops[1:]:
        bad = margin.small_margin_rows(oracle.gate_logits(ops["x"], ops["W_gate"], ops["bias"]), k, 1e-3)
        keep[bad] = False
    return shapes, all_ops, members, dev0["x"], np.nonzero(keep)[0]


@pytest.mark.parametrize("T,d_in,d_outs,N,r,k,routing,packed", [
    (33, 1024, (520, 136, 136), 28, 8, 2, "uniform", True),      # q/k/v-like, two launches for the group
    (64, 4096, (1032, 1032), 12, 16, 3, "zipf", True),           # gate/up-like, r = 16, bias
    (8, 512, (256, 264, 136, 72), 28, 8, 2, "uniform", True),    # four members
    (33, 512, (8200, 4104, 3080), 28, 8, 2, "uniform", True),    # 132 row tiles: runs that go on from member to member
    (5, 512, (16392, 8200, 8200), 28, 16, 2, "zipf", True),      # 274: runs longer than a row tile, two Wcat tiles cut
    (33, 1024, (520, 136), 28, 8, 2, "uniform", False),          # not packed: member by member
    (300, 512, (256, 264), 28, 8, 2, "uniform", True),           # a few hundred tokens: two launches with 160-row tiles
    (16, 512, (264,), 28, 8, 2, "zipf", True),                   # a group of one is the single-layer call
    (128, 1024, (520, 136, 136), 28, 8, 2, "uniform", True),     # q/k/v-like at T = 128
    (200, 1024, (776, 776), 12, 16, 3, "zipf", True),            # gate/up-like, r = 16, bias, ragged token tile
    (130, 512, (256, 264, 136, 72), 28, 8, 2, "uniform", True),  # four members: eight matrices in one launch
    (96, 768, (8200, 8192), 28, 8, 2, "uniform", True),          # 135 column tiles: two workgroups per CU
    (300, 512, (256, 264), 28, 8, 2, "uniform", False),          # a few hundred tokens, not packed: member by member
    (2000, 512, (2048, 2048, 2048), 28, 8, 2, "uniform", True),  # too many output tiles for one launch: member by member
], ids=["qkv", "gate-up-r16", "four", "runs", "long-runs", "unpacked", "T=300", "one", "qkv-T128", "gate-up-T200-r16", "four-T130",
        "T=96-two-per-CU", "T=300-unpacked", "T=2000"])
def test_group_call_matches_oracle_and_single_calls(T, d_in, d_outs, N, r, k, routing, packed):
    shapes, all_ops, members, x, rows = _group_case(T, d_in, d_outs, N, r, k, routing, seed=50)
    for mb in members:
        mb["packed"] = m.pack_weights(mb["W_gate"], mb["A"], mb["B"]) if packed else None
    res = m.linear_forward_group(x, members, k, 2.0, return_routing=True)
    torch.cuda.synchronize()
    for sh, ops, mb, (out, idx, w) in zip(shapes, all_ops, members, res):
        ref = oracle.linear_forward(ops["x"], ops["W"], ops["W_gate"], ops["bias"], ops["A"], ops["B"], k, 2.0)
        assert np.array_equal(_np(idx)[rows], ref["idx"][rows]), f"{sh.name}: routing differs from the oracle"
        assert np.all(np.abs(_np(w) - ref["w"])[rows] <= util.weight_bound(ops, ref["idx"])[rows])
        y = out.to(torch.float64).cpu().numpy()
        err = float(np.abs(y[rows] - ref["y"][rows]).max() / np.abs(ref["y"][rows]).max())
        assert err <= util.tol(sh), f"{sh.name}: rel err {err:.3e}"
        single, idx1, w1 = m.linear_forward(x, mb["W"], mb["W_gate"], mb["gate_bias"], mb["A"], mb["B"], k, 2.0,
                                            return_routing=True, packed=mb["packed"])
        assert torch.equal(idx[torch.from_numpy(rows).cuda()], idx1[torch.from_numpy(rows).cuda()])
        assert util.rel_max_err(out, single.to(torch.float64).cpu().numpy()) <= 2 * util.tol(sh)


# 64 adapters, 2048 -> 14336 twice: 260 column tiles and more.  The two-launch form lays out fp32 tiles and routing alone, which 24 MB
# hold; member by member the expand operands need more, and the outputs are those of the single calls bit for bit.
@pytest.mark.parametrize("T,k,r,two_launches", [(65, 4, 32, True), (120, 4, 32, True), (65, 8, 32, False), (68, 8, 32, False)])
def test_a_group_of_more_tiles_than_CUs(T, k, r, two_launches):
    d_in, d_out, N, bf = 2048, 14336, 64, torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(73)
    rand = lambda std, *shape: torch.randn(*shape, generator=g, device="cuda") * std
    x, members = rand(1.0, T, d_in).to(bf), []
    for _ in range(2):
        mb = {"W": rand(d_in ** -0.5, d_out, d_in).to(bf), "W_gate": rand(d_in ** -0.5, d_in, N), "gate_bias": None,
              "A": rand(d_in ** -0.5, N, d_in, r).to(bf), "B": rand(r ** -0.5, N, r, d_out).to(bf)}
        members.append(dict(mb, packed=m.pack_weights(mb["W_gate"], mb["A"], mb["B"])))
    small = torch.empty(24 << 20, dtype=torch.uint8, device="cuda")
    if two_launches:
        res = m.linear_forward_group(x, members, k, 0.5, ws=small, return_routing=True)
    else:
        with pytest.raises(m.MeteoraError):
            m.linear_forward_group(x, members, k, 0.5, ws=small)
        res = m.linear_forward_group(x, members, k, 0.5, return_routing=True)
    for mb, (out, idx, w) in zip(members, res):
        ref, idx1, w1 = m.linear_forward(x, mb["W"], mb["W_gate"], None, mb["A"], mb["B"], k, 0.5, return_routing=True, packed=mb["packed"])
        assert torch.equal(idx, idx1)
        if two_launches:   # one rounding of an fp32 sum each, the single call rounds s * w * h to bf16 as well
            assert util.rel_max_err(out, ref.to(torch.float64).cpu().numpy()) <= 2e-2
        else:
            assert torch.equal(out, ref) and torch.equal(w, w1)


# The tail's stretches of 512 columns, dealt to the XCDs where B is more than 4 MB: pairs of stretch and token that are no multiple of
# eight, fewer than eight, a short last stretch; both sides of 4 MB (18 and 19 stretches of 28 adapters of rank 8).
@pytest.mark.parametrize("T,d_in,d_out,N,r,k", [
    (1, 64, 2056, 64, 32, 4), (7, 136, 2056, 64, 32, 4), (64, 72, 2048, 64, 32, 2), (97, 1032, 2056, 64, 32, 2), (3, 64, 1032, 60, 36, 3),
    (1, 64, 520, 64, 64, 2), (5, 64, 9216, 28, 8, 2), (5, 64, 9224, 28, 8, 2), (70, 1024, 9224, 28, 8, 2), (1, 520, 16392, 28, 16, 8)])
def test_stretches_of_the_tail_by_xcd(T, d_in, d_out, N, r, k):
    assert _sequence(T, d_in, d_out, N, r, k) == ("decode" if T <= 64 else "few-tile")
    _check_layer(LS(T, d_in, d_out, N, r, k, 0.5 if r > 16 else 2.0, "bf16", "zipf", "stretches"), seed=74)


# ------------------------------------------------ temperature (App. A.6) and the top-1 strategy (App. A.1)
# one shape per launch sequence of the whole-layer call: decode (two launches), a few hundred tokens with the
# projection split along K, dense routing in front of the fused GEMM, the few-tile form again with rank 12, bucketed (2240 rows of
# Wcat), fp32
SEQUENCE_SHAPES = [
    LS(48, 1024, 520, 28, 8, 2, 2.0, "bf16", "uniform", "decode"),
    LS(200, 1024, 1096, 28, 8, 2, 2.0, "bf16", "zipf", "mid-split"),
    LS(2500, 512, 2056, 28, 8, 2, 2.0, "bf16", "uniform", "dense-route"),
    LS(700, 512, 264, 28, 12, 2, 2.0, "bf16", "zipf", "bucketed"),
    LS(1300, 320, 2056, 64, 32, 4, 0.5, "bf16", "zipf", "lists"),
    LS(90, 264, 136, 6, 8, 2, 2.0, "f32", "uniform", "fp32"),
]


@pytest.mark.parametrize("tau", [15.0, 20.0, 30.0])
@pytest.mark.parametrize("shape", SEQUENCE_SHAPES, ids=lambda s: s.name)
def test_linear_forward_with_temperature(shape, tau):
    """softmax(g / tau) over the selected logits in the whole-layer call (the reading of App. A.6; the formula is
    not printed in the paper): same adapters, weights and output as the oracle's with the same temperature."""
    _check_layer(shape, seed=51, inv_temperature=1.0 / tau)


@pytest.mark.parametrize("shape", SEQUENCE_SHAPES, ids=lambda s: s.name)
def test_linear_forward_top1(shape):
    """k = 1 (App. A.1): the weight is exactly 1 on every path, whatever the temperature, and the layer is
    x W + s (x A_a) B_a for the single best adapter a."""
    import dataclasses
    sh = dataclasses.replace(shape, k=1)
    _check_layer(sh, seed=52)
    ops, dev = util.make_case(sh, seed=52)
    y1, idx1, w1 = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], dev["bias"], dev["A"], dev["B"], 1, sh.scale,
                                    return_routing=True)
    y2, idx2, w2 = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], dev["bias"], dev["A"], dev["B"], 1, sh.scale,
                                    return_routing=True, inv_temperature=1.0 / 20.0)
    assert torch.equal(w1, torch.ones_like(w1)) and torch.equal(w2, w1)
    assert torch.equal(idx1, idx2) and torch.equal(y1, y2)


@pytest.mark.parametrize("missing", ["W_gate", "A", "B"])
def test_group_call_with_a_missing_tensor_is_refused_by_the_library(missing):
    """A member without one of its tensors: the library's invalid-argument status, as in the single-layer call."""
    _, _, members, x, _ = _group_case(33, 1024, (520, 136), 28, 8, 2, "uniform", seed=53)
    for mb in members:
        mb["packed"] = m.pack_weights(mb["W_gate"], mb["A"], mb["B"])
    members[1][missing] = None
    with pytest.raises(m.MeteoraError) as e:
        m.linear_forward_group(x, members, 2, 2.0)
    assert e.value.status == 1


def test_group_call_with_temperature():
    """The grouped call passes the temperature on to every member (decode-sized group, two launches)."""
    shapes, all_ops, members, x, rows = _group_case(33, 1024, (520, 136), 28, 8, 2, "uniform", seed=53)
    for mb in members:
        mb["packed"] = m.pack_weights(mb["W_gate"], mb["A"], mb["B"])
    res = m.linear_forward_group(x, members, 2, 2.0, return_routing=True, inv_temperature=1.0 / 15.0)
    torch.cuda.synchronize()
    for sh, ops, (out, idx, w) in zip(shapes, all_ops, res):
        ref = oracle.linear_forward(ops["x"], ops["W"], ops["W_gate"], ops["bias"], ops["A"], ops["B"], 2, 2.0,
                                    temperature=15.0)
        assert np.array_equal(_np(idx)[rows], ref["idx"][rows])
        assert np.all(np.abs(_np(w) - ref["w"])[rows] <= util.weight_bound(ops, ref["idx"], 1.0 / 15.0)[rows])
        y = out.to(torch.float64).cpu().numpy()
        assert float(np.abs(y[rows] - ref["y"][rows]).max() / np.abs(ref["y"][rows]).max()) <= util.tol(sh)


def test_init_then_first_call_inside_a_graph_capture():
    """meteora_init sets every kernel's LDS limit ahead of time, so a call can be captured without an eager call
    of the same kind before it (this process may have launched these kernels already; the call order is what a
    capturing caller uses)."""
    m.init()
    m.init(0)
    shape = LS(130, 1024, 520, 28, 8, 2, 2.0, "bf16", "uniform", "graph-after-init")
    ops, dev = util.make_case(shape, seed=54, condition=False)
    packed = m.pack_weights(dev["W_gate"], dev["A"], dev["B"])
    ws = torch.empty(m.workspace_bytes(shape.T, shape.d_in, shape.d_out, shape.N, shape.r, shape.k, torch.bfloat16),
                     dtype=torch.uint8, device="cuda")
    out = torch.empty((shape.T, shape.d_out), dtype=torch.bfloat16, device="cuda")
    args = (dev["x"], dev["W"], dev["W_gate"], dev["bias"], dev["A"], dev["B"], shape.k, shape.scale)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            m.linear_forward(*args, out=out, ws=ws, packed=packed)
    torch.cuda.synchronize()
    ref = m.linear_forward(*args, packed=packed)
    for _ in range(2):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)


def test_linear_forward_single_adapter_is_merged_gemm():
    """N=1,k=1: the layer is x(W + s*A*B) (Eq. 1)."""
    shape = LS(100, 256, 264, 1, 8, 1, 2.0, "f32")
    ops, dev = util.make_case(shape, seed=43, condition=False)
    y = m.linear_forward(dev["x"], dev["W"], dev["W_gate"], None, dev["A"], dev["B"], 1, 2.0)
    merged = ops["W"].astype(np.float64).T + 2.0 * ops["A"][0].astype(np.float64) @ ops["B"][0].astype(np.float64)
    assert util.rel_max_err(y, ops["x"].astype(np.float64) @ merged) <= 1e-5


# --------------------------------------------------- the seeded configurations at their full sizes
def test_config1_tiny_fp32_all_rows():
    seed, layers = gen.config_layers(1)
    _check_layer(layers[0], seed)


def test_config2_q_proj_prefill_sampled_rows():
    seed, layers = gen.config_layers(2)
    _check_layer(layers[0], seed, rows="sample")


def test_config4_decode_all_rows():
    seed, layers = gen.config_layers(4)
    for li, shape in enumerate(layers):
        _check_layer(shape, seed, li)


@pytest.mark.parametrize("li", [0, 1, 2])
def test_config3_mlp_zipf_sampled_rows(li):
    seed, layers = gen.config_layers(3)
    _check_layer(layers[li], seed, li, rows="sample")


@pytest.mark.parametrize("li", [0, 1, 2, 3, 4, 5, 6])
def test_config5_block_sampled_rows(li):
    seed, layers = gen.config_layers(5)
    _check_layer(layers[li], seed, li, rows="sample")
