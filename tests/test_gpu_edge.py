"""GPU parity on the degenerate inputs the method has (Section 1.1: smoothing, per-block INT8 scales, FP8
weights; Section 1.3: Top-K classification): operands whose quantisation scale is taken from an all-zero
block, rows of equal block scores, a key block that outweighs everything before it by more than the
rescaling hardware can express in one step, inputs of larger magnitude -- and the longest sequence the
library accepts.  Every case goes through the C ABI and is compared with the oracle like the ordinary cases."""
import numpy as np
import pytest
import torch

from oracle import sla_oracle as so
from paper_2512_16093_amd import binding as sla
from paper_2512_16093_amd import synth

import parity_util as pu

pytestmark = pytest.mark.gpu


def _constant_keys(q, k, v):
    """Every key the same vector: smoothing leaves all-zero keys (scale 1, codes 0), all scores and all
    pooled scores are equal (classification by index alone, uniform attention)."""
    k = k.clone()
    k[:] = k[0, 0, 0]
    return q, k, v


def _zero_blocks(q, k, v):
    """An all-zero query block (scale 1, scores 0, equal pooled scores), an all-zero and a constant channel of V
    (the first has scale 1 and codes 0), a key block that repeats one vector."""
    q, k, v = q.clone(), k.clone(), v.clone()
    q[:, :, :128] = 0
    v[..., 5] = 0
    v[..., 9] = 1.5
    k[:, :, 64:128] = k[:, :, 64:65]
    return q, k, v


def _late_dominant_block(q, k, v):
    """The last key block scores ~ 50 nats above everything before it for every query: the reference level
    jumps by more than 64 binary orders at the end of every row, beyond what one block scale expresses."""
    q, k = q.float(), k.float()
    q = q + 1.8
    N = k.shape[2]
    k[:, :, (N - 1) // 64 * 64:] += 2.4
    return q.to(torch.bfloat16), k.to(torch.bfloat16), v


def _doubled(q, k, v):
    """Q and K times two (exact in bf16): scores four times as large, sharper rows, more weights that round to 0."""
    return (q.float() * 2).to(torch.bfloat16), (k.float() * 2).to(torch.bfloat16), v


def _check_sharp_rows(gpu, ref, what):
    """The bar for inputs that make rows sharp (a few keys carry most of a row's weight).  There a single FP8
    weight (3 mantissa bits: relative step 2^-4 .. 2^-3) that rounds the other way in the kernel's fp32 than
    in the oracle's fp64 is worth several percent of the output, and the kernel knows a weight's exponent to
    ~1e-4 only (the score bias it carries through the conversion-free exponent costs that much).  Such rows are
    few and scattered; an indexing or scaling mistake moves most rows.  So: at most 1 % of the rows beyond the
    usual 2e-2, none beyond 8e-2, cosine as usual."""
    gpu = np.asarray(gpu, dtype=np.float64)
    assert np.isfinite(gpu).all(), what + ": non-finite output"
    row_err = np.abs(gpu - ref).max(axis=1)
    assert row_err.max() <= 8e-2, "%s: max-abs %.3e" % (what, row_err.max())
    assert (row_err > pu.MAX_ABS).mean() <= 0.01, "%s: %d rows beyond %.0e" % (what, (row_err > pu.MAX_ABS).sum(), pu.MAX_ABS)
    assert pu.cosine(gpu, ref) >= pu.MIN_COS, what + ": cosine"


CASES = {"constant_keys": _constant_keys, "zero_blocks": _zero_blocks, "late_dominant_block": _late_dominant_block,
         "doubled": _doubled}


@pytest.mark.parametrize("bq", [128, 64])
@pytest.mark.parametrize("name", sorted(CASES))
def test_degenerate_inputs_low_bit_forward(name, bq):
    cfg = synth.custom_config(1, 2, (5, 10, 20), block_q=bq, topk_ratio=0.25, marginal_ratio=0.5, cfg_id=700)
    q, k, v = CASES[name](*synth.make_qkv(cfg))
    W = synth.make_proj(cfg)
    qd, kd, vd, Wd = pu.to_dev(q, k, v, W)
    out = sla.sla_attention_fwd(qd, kd, vd, bq, 64, cfg.topk_ratio, cfg.marginal_ratio, proj_w=Wd).float().cpu().numpy()
    mask = sla.sla_classify_blocks(qd, kd, bq, 64, cfg.topk_ratio, cfg.marginal_ratio)[0].cpu().numpy()
    Tq, Tk, n_c, n_m = so.block_counts(cfg.N, bq, 64, cfg.topk_ratio, cfg.marginal_ratio)
    assert np.isfinite(out).all()
    qc, qs = (t.cpu().numpy() for t in sla.sla_debug_quantize_q(qd, bq))
    vc = sla.sla_debug_quantize_kv(kd, vd)[3].cpu().numpy()
    from oracle import formats
    for h in range(cfg.H):
        # the operands quantised from 16-bit inputs carry the oracle's codes exactly (zero blocks and exact ties included)
        Q8, dq = so.quantize_q(synth.as_f64(q[0, h]), bq)
        assert np.array_equal(qc[0, h].astype(np.float64), Q8) and np.allclose(qs[0, h], dq, rtol=1e-6)
        assert np.array_equal(formats.e4m3_decode(vc[0, h]), so.quantize_v(synth.as_f64(v[0, h]))[0])
        r = pu.oracle_head(cfg, q, k, v, 0, h, W)
        nbad, _, _ = pu.check_mask(mask[0, h], r["scores"], n_c, n_m, "%s head %d" % (name, h))
        if nbad:
            r = pu.oracle_head(cfg, q, k, v, 0, h, W, mask=mask[0, h])
        if name in ("doubled", "late_dominant_block"):
            _check_sharp_rows(out[0, h], r["out"], "%s head %d" % (name, h))
        else:
            pu.check_output(out[0, h], r["out"], "%s head %d" % (name, h))
    if name == "constant_keys":   # equal scores everywhere: the lowest block indices win, in every row
        assert (mask[..., :n_c] == 1).all() and (mask[..., n_c:n_c + n_m] == 0).all() and (mask[..., n_c + n_m:] == -1).all()


@pytest.mark.parametrize("bq", [128, 64])
@pytest.mark.parametrize("name", sorted(CASES))
def test_degenerate_inputs_unquantised_forward_and_backward(name, bq):
    """The same inputs through the 16-bit forward pass (steps of two key tiles and of one) and the backward pass (bf16
    products, fp32 statistics)."""
    from oracle import sla_bwd_oracle as bo
    cfg = synth.custom_config(1, 1, (5, 10, 20), block_q=bq, topk_ratio=0.25, marginal_ratio=0.5, cfg_id=701)
    q, k, v = CASES[name](*synth.make_qkv(cfg))
    W = synth.make_proj(cfg)
    dout = synth.make_qkv(cfg, seed=5)[2]
    qd, kd, vd, Wd, dd = pu.to_dev(q, k, v, W, dout)
    out = sla.sla_attention_fwd(qd, kd, vd, bq, 64, cfg.topk_ratio, cfg.marginal_ratio, proj_w=Wd,
                                quant_mode=sla.QUANT_NONE).float().cpu().numpy().astype(np.float64)
    mask = sla.sla_classify_blocks(qd, kd, bq, 64, cfg.topk_ratio, cfg.marginal_ratio, want_scores=False)[0].cpu().numpy()
    Q, K, V, D = (synth.as_f64(t[0, 0]) for t in (q, k, v, dout))
    r = so.sla_forward_head(Q, K, V, bq, 64, cfg.topk_ratio, cfg.marginal_ratio, proj_w=synth.as_f64(W),
                            quant=so.QUANT_NONE, mask=mask[0, 0])
    pu.check_output(out[0, 0], r["out"], name + " unquantised forward")
    g = sla.sla_attention_bwd(qd, kd, vd, dd, bq, 64, cfg.topk_ratio, cfg.marginal_ratio, proj_w=Wd)
    ref = bo.sla_backward_head(Q, K, V, D, mask[0, 0], bq, 64, proj_w=synth.as_f64(W), has_bias=False)
    for key, got in (("dQ", g[0]), ("dK", g[1]), ("dV", g[2])):
        a = got[0, 0].float().cpu().numpy().astype(np.float64)
        b = ref[key]
        assert np.isfinite(a).all(), "%s %s: non-finite" % (name, key)
        # (with constant keys dQ is exactly 0 -- the rows of dS sum to zero -- and the bf16 path leaves rounding
        # residue of dS times |K| there: the bounds are taken relative to a magnitude of at least 1)
        scale = max(np.abs(b).max(), 1.0)
        assert np.linalg.norm(a - b) <= 1e-2 * max(np.linalg.norm(b), np.sqrt(b.size)), "%s %s: Frobenius" % (name, key)
        assert np.abs(a - b).max() <= 3e-2 * scale, "%s %s: element" % (name, key)


@pytest.mark.parametrize("bq", [128, 64])
@pytest.mark.parametrize("n_c", [2, 5, 6, 7, 8, 9, 17])
def test_every_list_length_through_the_sparse_stage(n_c, bq):
    """The attention kernel's main loop takes four list entries per round, up to three more one by one, and the
    ragged last key block apart: lists of every remainder, with and without the last block, chosen at random
    (ascending, as the classification delivers them), through sla_sparse_attn_fwd against the oracle on the same mask.
    With query blocks of 64 the loop takes two entries per round and its copy rings are shorter."""
    cfg = synth.custom_config(1, 2, (6, 7, 25), block_q=bq, topk_ratio=0.2, marginal_ratio=0.4, cfg_id=710)   # N = 1050, Tk = 17
    q, k, v = synth.make_qkv(cfg)
    Tq, Tk = -(-cfg.N // bq), -(-cfg.N // 64)
    rng = np.random.default_rng(1000 * n_c + bq)
    masks = np.full((1, cfg.H, Tq, Tk), -1, dtype=np.int8)
    for h in range(cfg.H):
        for i in range(Tq):
            pick = rng.choice(Tk, size=n_c, replace=False)
            if i % 3 == 0 and (Tk - 1) not in pick:      # a third of the rows must end in the ragged block
                pick[0] = Tk - 1
            if i % 3 == 1 and n_c < Tk:                  # a third must not
                pick = rng.choice(Tk - 1, size=n_c, replace=False)
            masks[0, h, i, pick] = 1
    crit = pu.lists_from_mask(masks)
    out, lse = sla.sla_sparse_attn_fwd(*pu.to_dev(q, k, v, crit), bq, 64)
    out, lse = out.cpu().numpy(), lse.cpu().numpy()
    for h in range(cfg.H):
        ref, ref_lse = so.sparse_branch_quant(synth.as_f64(q[0, h]), synth.as_f64(k[0, h]), synth.as_f64(v[0, h]),
                                              masks[0, h], bq, 64, return_lse=True, ref_tile=pu.REF_TILE)
        pu.check_output(out[0, h], ref, "n_c %d head %d" % (n_c, h))
        dl = np.abs(lse[0, h] - ref_lse)
        assert dl.max() < 2e-2 and np.median(dl) < 1e-5


@pytest.mark.parametrize("quant", [sla.QUANT_QK_INT8_PV_FP8, sla.QUANT_NONE])
@pytest.mark.parametrize("bq", [128, 64])
@pytest.mark.parametrize("n_c", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11])
def test_every_list_length_with_the_linear_branch(n_c, bq, quant):
    """The summaries of a query block take the places of the staged key blocks behind the end of its list (which place
    depends on the list's length and on whether it ends in the ragged block); bias and result start at any element."""
    cfg = synth.custom_config(1, 2, (6, 7, 25), block_q=bq, topk_ratio=n_c / 17, marginal_ratio=4 / 17, cfg_id=711)   # N = 1050, Tk = 17
    q, k, v = synth.make_qkv(cfg, seed=n_c)
    W, bias = synth.make_proj(cfg), synth.make_qkv(cfg, seed=3)[0][0, 0, 0].contiguous()
    odd = torch.zeros(129, dtype=torch.bfloat16, device="cuda")
    odd[1:] = bias.cuda()
    out = torch.empty(q.numel() + 1, dtype=torch.bfloat16, device="cuda")[1:].view(q.shape)
    args = (bq, 64, cfg.topk_ratio, cfg.marginal_ratio)
    sla.sla_attention_fwd(*pu.to_dev(q, k, v), *args, proj_w=W.cuda(), proj_b=odd[1:], quant_mode=quant, out=out)
    mask = sla.sla_classify_blocks(*pu.to_dev(q, k), *args, want_scores=False)[0].cpu().numpy()
    assert ((mask == 1).sum(-1) == n_c).all() and (mask[..., -1] == 1).any() and (mask[..., -1] != 1).any()   # both kinds of end
    for h in range(cfg.H):
        ref = so.sla_forward_head(*(synth.as_f64(x[0, h]) for x in (q, k, v)), *args, proj_w=synth.as_f64(W),
                                  proj_b=synth.as_f64(bias), mask=mask[0, h], ref_tile=pu.REF_TILE,
                                  quant=so.QUANT_NONE if quant == sla.QUANT_NONE else so.QUANT_QK_INT8_PV_FP8)["out"]
        got = out[0, h].float().cpu().numpy().astype(np.float64)
        pu.check_output(got, ref, "n_c %d head %d" % (n_c, h))
        # (bf16 results: 1.7e-3 of rounding; 5e-3 as in the parity tests)
        assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 5e-3


@pytest.mark.parametrize("grid", [(6, 7, 25), (1, 8, 24), (2, 8, 8), (1, 5, 5)])   # 17 (ragged), 3, 2 and 1 query blocks
def test_all_critical_blocks_of_64_queries_share_a_workgroup(grid):
    """Every key block critical at query blocks of 64: two adjacent blocks then share one walk over the records.
    The stage entry point (which takes any lists) walks them one by one: the same arithmetic, so the same bits."""
    cfg = synth.custom_config(1, 2, grid, block_q=64, topk_ratio=1.0, marginal_ratio=0.0, cfg_id=740)
    q, k, v = pu.to_dev(*synth.make_qkv(cfg))
    Tk = -(-cfg.N // 64)
    crit = torch.arange(Tk, dtype=torch.int32, device="cuda").repeat(1, cfg.H, Tk, 1).contiguous()
    out = sla.sla_attention_fwd(q, k, v, 64, 64, 1.0, 0.0)
    stage, _ = sla.sla_sparse_attn_fwd(q, k, v, crit, 64, 64)
    assert torch.equal(out, stage.to(torch.bfloat16))


def test_codes_of_blocks_with_tiny_maxima():
    """Blocks whose largest magnitude is far below the reciprocal's range (16-bit inputs reach 2^-133; 1 / 2^-130
    overflows fp32): the quotient is formed on a rescaled maximum, the codes are still the oracle's."""
    from oracle import formats
    cfg = synth.custom_config(1, 1, (2, 8, 16), block_q=128, topk_ratio=0.5, marginal_ratio=0.5, cfg_id=730)   # N = 256
    q, k, v = synth.make_qkv(cfg)
    q, v = q.float(), v.float()
    q[:, :, :128] *= 2.0 ** -128          # first query block: maxima near 2^-126, most values denormal in bf16
    v[..., 3] *= 2.0 ** -127
    v[..., 7] *= 2.0 ** -110
    q, v = q.to(torch.bfloat16), v.to(torch.bfloat16)
    qc, qs = (t.cpu().numpy() for t in sla.sla_debug_quantize_q(q.cuda(), 128))
    vc = sla.sla_debug_quantize_kv(k.cuda(), v.cuda())[3].cpu().numpy()
    Q8, dq = so.quantize_q(synth.as_f64(q[0, 0]), 128)
    assert np.array_equal(qc[0, 0].astype(np.float64), Q8) and np.allclose(qs[0, 0], dq, rtol=1e-6)
    assert np.array_equal(formats.e4m3_decode(vc[0, 0]), so.quantize_v(synth.as_f64(v[0, 0]))[0])
    out = sla.sla_attention_fwd(q.cuda(), k.cuda(), v.cuda(), 128, 64, 0.5, 0.5).float().cpu().numpy()
    r = pu.oracle_head(cfg, q, k, v, 0, 0, None)
    pu.check_output(out[0, 0], r["out"], "tiny maxima")


@pytest.mark.parametrize("N", [40, 1050, 4096, 4097, 4160, 12790])   # 1, 17 (ragged), 64, 65 (one key), 65 and 200 (ragged) key blocks
def test_mean_of_k_keeps_its_order_of_summation(N):
    """The INT8 codes of K hang on the last bit of its channel mean, so the order in which the mean is summed is part of
    the result: 64 interleaved partial sums over the key blocks, then those in ascending order, all in fp32.  Keys that
    are constant within a block (block means are then exact) make the sum reproducible on the host, bit for bit."""
    rng = np.random.default_rng(N)
    Tk = -(-N // 64)
    rows = torch.from_numpy(rng.standard_normal((2, Tk, 128)) * 2.0 ** rng.integers(-6, 7, (2, Tk, 1))).to(torch.bfloat16)
    k = rows.repeat_interleave(64, 1)[None, :, :N].contiguous().cuda()
    mean = sla.sla_debug_quantize_kv(k, k)[2].cpu().numpy()[0]
    count = np.minimum(64, N - 64 * np.arange(Tk)).astype(np.float32)
    share = rows.float().numpy() * count[None, :, None]            # (exact: eight bits times at most 64)
    runs = np.zeros((2, 64, 128), np.float32)
    for j in range(Tk):
        runs[:, j % 64] += share[:, j]
    total = np.zeros((2, 128), np.float32)
    for r in range(64):
        total += runs[:, r]
    assert np.array_equal(mean.view(np.int32), (total / np.float32(N)).view(np.int32))


@pytest.mark.parametrize("bq", [128, 64])
def test_linear_term_of_query_tokens_of_any_magnitude(bq):
    """softmax in phi(Q) subtracts a token's maximum before anything is scaled: at every finite magnitude its largest channel has
    the largest weight, in the low-bit kernel (the stage alone: no INT8 scores of such tokens) and in the unquantised forward
    pass (keys of 1e-36: its scores stay in range)."""
    cfg = synth.custom_config(1, 2, (5, 10, 20), block_q=bq, topk_ratio=0.25, marginal_ratio=0.5, cfg_id=712)   # N = 1000
    q, k, v = synth.make_qkv(cfg)
    rng = np.random.default_rng(bq)
    size = 10.0 ** rng.uniform(0, 30, (1, cfg.H, cfg.N, 1))
    size[:, :, 7::bq] = 2.0 ** rng.uniform(126, 127.99, size[:, :, 7::bq].shape)   # one token per query block (its mean has to stay finite)
    q = torch.from_numpy(rng.uniform(-1, 1, q.shape) * size).to(torch.bfloat16)
    W = synth.make_proj(cfg)
    args = (bq, 64, cfg.topk_ratio, cfg.marginal_ratio)
    for name, keys in (("stage", k), ("unquantised", (k.float() * 1e-36).to(torch.bfloat16))):
        qd, kd, vd, Wd = pu.to_dev(q, keys, v, W)
        if name == "stage":
            mask = torch.from_numpy(rng.integers(-1, 2, (1, cfg.H, -(-cfg.N // bq), -(-cfg.N // 64)), dtype=np.int8)).cuda()
            out = sla.sla_linear_attn_fwd(qd, kd, vd, mask, bq, 64, proj_w=Wd)
        else:
            mask = sla.sla_classify_blocks(qd, kd, *args, want_scores=False)[0]
            out = sla.sla_attention_fwd(qd, kd, vd, *args, proj_w=Wd, quant_mode=sla.QUANT_NONE)
        for h in range(cfg.H):
            Q, K, V = (synth.as_f64(x[0, h]) for x in (q, keys, v))
            m = mask[0, h].cpu().numpy()
            if name == "stage":
                ref = so.linear_branch(Q, K, V, m, bq, 64) @ synth.as_f64(W).T
            else:
                ref = so.sla_forward_head(Q, K, V, *args, proj_w=synth.as_f64(W), quant=so.QUANT_NONE, mask=m)["out"]
            got = out[0, h].float().cpu().numpy().astype(np.float64)
            pu.check_output(got, ref, "%s head %d" % (name, h))
            # (bf16 results and summaries: 1.7e-3 of rounding each; 5e-3 as in the parity tests)
            assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 5e-3, name


@pytest.mark.parametrize("bq", [128, 64])
def test_linear_term_of_values_near_the_largest(bq):
    """phi(Q) sums to at most 1 over the channels when it meets H_i: what the quotient leaves finite does not overflow ahead of it.
    768 values of 6e35 under flat weights: H_i holds 3.6e36 per channel, of which 128 channels of weight 0.95 would make 4.4e38.
    (Not larger: V's quantisation takes 448 times a value.)"""
    cfg = synth.custom_config(1, 1, (4, 16, 16), block_q=bq, topk_ratio=0.25, marginal_ratio=0.75, cfg_id=713)   # N = 1024
    q, k, v = synth.make_qkv(cfg)
    q, k = ((x.float() / 64).to(torch.bfloat16) for x in (q, k))
    v = ((1.0 + 0.1 * v.float().clamp(-2, 2)) * 6e35).to(torch.bfloat16)
    qd, kd, vd = pu.to_dev(q, k, v)
    args = (bq, 64, cfg.topk_ratio, cfg.marginal_ratio)
    mask = sla.sla_classify_blocks(qd, kd, *args, want_scores=False)[0]
    m = mask[0, 0].cpu().numpy()
    Q, K, V = (synth.as_f64(x[0, 0]) for x in (q, k, v))
    got = {"stage": sla.sla_linear_attn_fwd(qd, kd, vd, mask, bq, 64)}
    want = {"stage": so.linear_branch(Q, K, V, m, bq, 64)}
    for name, quant, oq in (("unquantised", sla.QUANT_NONE, so.QUANT_NONE),
                            ("low-bit", sla.QUANT_QK_INT8_PV_FP8, so.QUANT_QK_INT8_PV_FP8)):
        got[name] = sla.sla_attention_fwd(qd, kd, vd, *args, quant_mode=quant)
        want[name] = so.sla_forward_head(Q, K, V, *args, mask=m, quant=oq, ref_tile=pu.REF_TILE)["out"]
    for name in got:
        x = got[name][0, 0].float().cpu().numpy().astype(np.float64)
        assert np.isfinite(x).all(), name
        # (as above; of the low-bit core's FP8 weights and values, flat here, 448 levels are left: 1e-2)
        assert np.linalg.norm(x - want[name]) / np.linalg.norm(want[name]) <= (1e-2 if name == "low-bit" else 5e-3), name
