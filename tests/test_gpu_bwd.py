"""GPU parity of the SLA backward pass: sla_attention_bwd (through the C ABI) against the float64
gradient oracle, element by element, on seeded synthetic inputs that span several tiles and ragged
tails.  The block mask is the library's own (its agreement with the oracle's classification is the
subject of the forward parity tests), so ties in the Top-K choice play no role here.

Tolerance.  The path computes in bf16 with fp32 accumulation: inputs are bf16 already; P, dS, the
per-block summaries H, Z, their gradients and the outputs are each rounded to bf16 once (relative
step 2^-9), the softmax statistics, delta and the normalisers stay in fp32.  A handful of
independent roundings of relative size 2^-9 per contribution, averaged over long sums, give a
relative Frobenius error well under 1e-2; single elements are held to 3e-2 of the largest
reference entry, and the direction (cosine) to 0.999 as for the forward pass."""
import numpy as np
import pytest
import torch

from oracle import sla_bwd_oracle as bo
from oracle import sla_oracle as so
from paper_2512_16093_amd import binding as sla
from paper_2512_16093_amd import synth

pytestmark = pytest.mark.gpu

REL_FRO, REL_MAX, COS_MIN = 1e-2, 3e-2, 0.999

CASES = [
    # (H, grid, block_q, rc, rm, proj)  -- batch 1; a batch of 2 is in test_backward_batch_of_two
    (2, (5, 10, 20), 128, 0.25, 0.0, False),   # sparse branch alone, N = 1000 (ragged in both block sizes)
    (2, (5, 10, 20), 64, 0.2, 0.0, False),
    (2, (5, 10, 20), 128, 0.25, 0.5, True),    # both branches with projection and bias gradient
    (2, (5, 10, 20), 64, 0.2, 0.4, True),
    (1, (3, 27, 27), 128, 0.1, 0.2, False),    # N = 2187 = 17*128 + 11, no projection (identity)
    (1, (1, 9, 9), 128, 0.5, 0.5, True),       # N = 81: one ragged query block, two key blocks
    (1, (1, 5, 5), 64, 1.0, 0.0, False),       # N = 25: a single short block, dense attention
    (1, (4, 16, 16), 64, 0.15, 0.85, True),    # N = 1024: whole blocks, no negligible block
    (2, (5, 10, 20), 128, 0.75, 0.25, True),   # most blocks critical: the dK/dV kernel's two-key-block variant
    (1, (3, 27, 27), 64, 0.6, 0.0, False),     # the same with an odd number of key blocks (35) and no linear term
]


def _compare(name, got, ref):
    got, ref = got.astype(np.float64), ref.astype(np.float64)
    scale = np.abs(ref).max()
    assert np.isfinite(got).all(), name
    if scale == 0.0:
        assert not got.any(), name
        return
    err = np.abs(got - ref).max()
    fro = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    cos = float((got * ref).sum() / np.linalg.norm(got) / np.linalg.norm(ref))
    assert err <= REL_MAX * scale and fro <= REL_FRO and cos >= COS_MIN, (name, err / scale, fro, cos)


@pytest.mark.parametrize("H,grid,bq,rc,rm,proj", CASES)
def test_backward_matches_gradient_oracle(H, grid, bq, rc, rm, proj):
    cfg = synth.custom_config(1, H, grid, block_q=bq, topk_ratio=rc, marginal_ratio=rm, use_proj=proj, cfg_id=300)
    q, k, v = synth.make_qkv(cfg)
    dout = synth.make_qkv(cfg, seed=7)[2]          # a V-like tensor as the upstream gradient
    W = synth.make_proj(cfg) if proj else None
    dev = torch.device("cuda:0")
    qd, kd, vd, dd = (t.to(dev) for t in (q, k, v, dout))
    Wd = W.to(dev) if proj else None
    print("case", H, grid, bq, rc, rm, proj, flush=True)
    mask = sla.sla_classify_blocks(qd, kd, bq, 64, rc, rm, want_scores=False)[0].cpu().numpy()
    dq, dk, dv, dw, db = sla.sla_attention_bwd(qd, kd, vd, dd, bq, 64, rc, rm, proj_w=Wd, want_dw=proj, want_db=proj)
    torch.cuda.synchronize()
    sums_w = np.zeros((cfg.d, cfg.d))
    sums_b = np.zeros(cfg.d)
    for h in range(H):
        r = bo.sla_backward_head(synth.as_f64(q[0, h]), synth.as_f64(k[0, h]), synth.as_f64(v[0, h]),
                                 synth.as_f64(dout[0, h]), mask[0, h], bq, 64,
                                 proj_w=synth.as_f64(W) if proj else None, has_bias=proj)
        _compare("dq", dq[0, h].float().cpu().numpy(), r["dQ"])
        _compare("dk", dk[0, h].float().cpu().numpy(), r["dK"])
        _compare("dv", dv[0, h].float().cpu().numpy(), r["dV"])
        if proj:
            sums_w += r["dW"]
            sums_b += r["db"]
    if proj:
        _compare("dproj_w", dw.cpu().numpy(), sums_w)
        _compare("dproj_b", db.cpu().numpy(), sums_b)


@pytest.mark.parametrize("N", [95, 97, 127, 161, 351])
def test_linear_branch_at_the_edges_of_its_token_tiles(N):
    """Query blocks of 64 in the linear branch: a wavefront pair owns 32 tokens, each half of the channels.  The last
    block holds a tile less one token, a tile and one, all but one; same bounds as above.  (One token: next test.)"""
    test_backward_matches_gradient_oracle(2, (1, 1, N), 64, 0.5, 0.5, True)


def _lone_key_bound(Q, K, V, dO, W, mask):
    """How far the roundings of the linear branch's bf16 operands move dK of the sequence's last key, if it is alone in its
    block: an array over the channels.

    d phi(K)[c] = sum_o G[c][o] V[o] + dZ[c].  Where that key is all a query block holds as marginal, O^l is its V whatever
    Q is, so the two terms cancel exactly, however large they are; what the roundings leave of them is the result.  Between
    the inputs and G V stand seven (phi(K), h, H, phi(Q), dnum, dH, G), independent from output channel to output channel, to
    dZ five (z, Z, phi(Q), dZ of a block, their sum).  A rounding is off by up to 2^-9, evenly spread: four standard
    deviations of the sum, then through the softmax, dK = phi o (d phi - phi . d phi)."""
    j = mask.shape[1] - 1
    qs, PQ, PK = so.block_slices(len(Q), 64), so.feature_map(Q, "softmax"), so.feature_map(K, "softmax")
    h, z = so.linear_summaries(K, V, 64, "softmax")
    G, dZ = np.zeros((128, 128)), np.zeros(128)
    for i in np.flatnonzero(mask[:, j] == 0):
        marg, a = np.flatnonzero(mask[i] == 0), PQ[qs[i]]
        den, dOl = a @ z[marg].sum(0), dO[qs[i]] @ W
        G += a.T @ (dOl / den[:, None])
        dZ -= a.T @ ((dOl * (a @ h[marg].sum(0))).sum(1) / den ** 2)
    sigma = 2.0 ** -9 / 3 ** 0.5 * np.sqrt(7 * ((G * V[-1]) ** 2).sum(1) + 5 * dZ ** 2)
    return 4 * PK[-1] * (sigma + np.sqrt(((PK[-1] * sigma) ** 2).sum()))


@pytest.mark.parametrize("N", [65, 129])
def test_gradient_of_a_key_alone_in_its_block(N):
    """The last block holds one token.  Every gradient but the lone key's dK is held to the bounds above.  That one may be
    what is left of sums that cancel (1000 and 2000 here, where the largest entry of dK is 1.5 and 1.2): 8 % and 18 % of the
    largest entry off with the bf16 summaries that the branch keeps, which the bound of `_lone_key_bound` allows for."""
    cfg = synth.custom_config(1, 2, (1, 1, N), block_q=64, topk_ratio=0.5, marginal_ratio=0.5, use_proj=True, cfg_id=300)
    q, k, v = synth.make_qkv(cfg)
    dout, W = synth.make_qkv(cfg, seed=7)[2], synth.make_proj(cfg)
    dev = [t.cuda() for t in (q, k, v, dout)]
    mask = sla.sla_classify_blocks(dev[0], dev[1], 64, 64, 0.5, 0.5, want_scores=False)[0].cpu().numpy()
    dq, dk, dv, dw, db = sla.sla_attention_bwd(*dev, 64, 64, 0.5, 0.5, proj_w=W.cuda(), want_dw=True, want_db=True)
    sums_w, sums_b, lone = 0.0, 0.0, 0
    for h in range(2):
        x, Wf = [synth.as_f64(t[0, h]) for t in (q, k, v, dout)], synth.as_f64(W)
        r = bo.sla_backward_head(*x, mask[0, h], 64, 64, proj_w=Wf, has_bias=True)
        gk = dk[0, h].float().cpu().numpy().astype(np.float64)
        _compare("dq", dq[0, h].float().cpu().numpy(), r["dQ"])
        _compare("dk", gk[:-1], r["dK"][:-1])
        _compare("dv", dv[0, h].float().cpu().numpy(), r["dV"])
        bound = _lone_key_bound(*x, Wf, mask[0, h])
        lone += int((mask[0, h, :, -1] == 0).any())
        err, scale = np.abs(gk[-1] - r["dK"][-1]), np.abs(r["dK"]).max()
        print("N %d head %d: lone key's dK off by %.3f of the largest entry, %.2f of its bound" % (
            N, h, err.max() / scale, (err / (bound + REL_MAX * scale)).max()), flush=True)
        assert (err <= bound + REL_MAX * scale).all()
        sums_w, sums_b = sums_w + r["dW"], sums_b + r["db"]
    assert lone                                        # (a head in which the lone key is marginal)
    _compare("dproj_w", dw.cpu().numpy(), sums_w)
    _compare("dproj_b", db.cpu().numpy(), sums_b)


@pytest.mark.parametrize("phi", ["elu1", "relu"])
@pytest.mark.parametrize("H,grid,bq,rc,rm", [(2, (5, 10, 20), 128, 0.25, 0.5), (1, (3, 27, 27), 64, 0.1, 0.9),
                                             (2, (5, 10, 20), 64, 0.75, 0.25)])
def test_backward_with_the_other_feature_maps(H, grid, bq, rc, rm, phi):
    """phi = elu + 1 or relu in the linear branch (the forward pass offers them; the oracle's gradient for
    them is pinned by the same finite-difference and autograd checks as the softmax's -- relu's on inputs
    kept away from its kink; the bf16 inputs here hold no exact zero that both sides would not treat
    alike, x > 0): both dK/dV variants."""
    cfg = synth.custom_config(1, H, grid, block_q=bq, topk_ratio=rc, marginal_ratio=rm, use_proj=True, cfg_id=303)
    q, k, v = synth.make_qkv(cfg)
    dout = synth.make_qkv(cfg, seed=11)[2]
    W = synth.make_proj(cfg)
    dev = torch.device("cuda:0")
    qd, kd, vd, dd, Wd = (t.to(dev) for t in (q, k, v, dout, W))
    mask = sla.sla_classify_blocks(qd, kd, bq, 64, rc, rm, want_scores=False)[0].cpu().numpy()
    dq, dk, dv, dw, db = sla.sla_attention_bwd(qd, kd, vd, dd, bq, 64, rc, rm, proj_w=Wd, want_dw=True, want_db=True,
                                               phi_kind=sla.PHI_ELU1 if phi == "elu1" else sla.PHI_RELU)
    torch.cuda.synchronize()
    sums_w, sums_b = np.zeros((cfg.d, cfg.d)), np.zeros(cfg.d)
    for h in range(H):
        r = bo.sla_backward_head(synth.as_f64(q[0, h]), synth.as_f64(k[0, h]), synth.as_f64(v[0, h]),
                                 synth.as_f64(dout[0, h]), mask[0, h], bq, 64, proj_w=synth.as_f64(W), has_bias=True,
                                 phi=phi)
        _compare("dq", dq[0, h].float().cpu().numpy(), r["dQ"])
        _compare("dk", dk[0, h].float().cpu().numpy(), r["dK"])
        _compare("dv", dv[0, h].float().cpu().numpy(), r["dV"])
        sums_w += r["dW"]
        sums_b += r["db"]
    _compare("dproj_w", dw.cpu().numpy(), sums_w)
    _compare("dproj_b", db.cpu().numpy(), sums_b)


def test_backward_batch_of_two():
    """Two batch entries with different contents: every (b, h) slice matches the oracle, and the
    projection gradients sum over both."""
    H, grid, bq, rc, rm = 2, (3, 9, 11), 128, 0.3, 0.5          # N = 297: ragged, Tq = 3 (odd), Tk = 5 (odd)
    cfg = synth.custom_config(2, H, grid, block_q=bq, topk_ratio=rc, marginal_ratio=rm, use_proj=True, cfg_id=301)
    q, k, v = synth.make_qkv(cfg)
    dout = synth.make_qkv(cfg, seed=9)[2]
    W = synth.make_proj(cfg)
    dev = torch.device("cuda:0")
    qd, kd, vd, dd, Wd = (t.to(dev) for t in (q, k, v, dout, W))
    assert not torch.equal(q[0], q[1])
    mask = sla.sla_classify_blocks(qd, kd, bq, 64, rc, rm, want_scores=False)[0].cpu().numpy()
    dq, dk, dv, dw, db = sla.sla_attention_bwd(qd, kd, vd, dd, bq, 64, rc, rm, proj_w=Wd, want_dw=True, want_db=True)
    torch.cuda.synchronize()
    sums_w, sums_b = np.zeros((cfg.d, cfg.d)), np.zeros(cfg.d)
    for b in range(2):
        for h in range(H):
            r = bo.sla_backward_head(synth.as_f64(q[b, h]), synth.as_f64(k[b, h]), synth.as_f64(v[b, h]),
                                     synth.as_f64(dout[b, h]), mask[b, h], bq, 64, proj_w=synth.as_f64(W), has_bias=True)
            _compare("dq", dq[b, h].float().cpu().numpy(), r["dQ"])
            _compare("dk", dk[b, h].float().cpu().numpy(), r["dK"])
            _compare("dv", dv[b, h].float().cpu().numpy(), r["dV"])
            sums_w += r["dW"]
            sums_b += r["db"]
    _compare("dproj_w", dw.cpu().numpy(), sums_w)
    _compare("dproj_b", db.cpu().numpy(), sums_b)


@pytest.mark.parametrize("H,grid,bq,rc,rm", [(2, (5, 10, 20), 128, 0.25, 0.5), (2, (3, 9, 11), 64, 0.3, 0.4)])
def test_backward_from_the_forward_pass_saved_state(H, grid, bq, rc, rm):
    """sla_attention_fwd_train gives the same output as the unquantised forward and a state with which
    sla_attention_bwd_saved matches the oracle to the same bar as the self-contained backward (and
    agrees with it closely: the only difference is delta formed from the bf16 O^s)."""
    cfg = synth.custom_config(1, H, grid, block_q=bq, topk_ratio=rc, marginal_ratio=rm, use_proj=True, cfg_id=302)
    q, k, v = synth.make_qkv(cfg)
    dout = synth.make_qkv(cfg, seed=5)[2]
    W = synth.make_proj(cfg)
    dev = torch.device("cuda:0")
    qd, kd, vd, dd, Wd = (t.to(dev) for t in (q, k, v, dout, W))
    out, saved = sla.sla_attention_fwd_train(qd, kd, vd, bq, 64, rc, rm, proj_w=Wd)
    ref_out = sla.sla_attention_fwd(qd, kd, vd, bq, 64, rc, rm, proj_w=Wd, quant_mode=sla.QUANT_NONE)
    assert torch.equal(out, ref_out)
    mask = sla.sla_classify_blocks(qd, kd, bq, 64, rc, rm, want_scores=False)[0].cpu().numpy()
    a = sla.sla_attention_bwd(qd, kd, vd, dd, bq, 64, rc, rm, proj_w=Wd, want_dw=True, want_db=True, saved=saved)
    b = sla.sla_attention_bwd(qd, kd, vd, dd, bq, 64, rc, rm, proj_w=Wd, want_dw=True, want_db=True)
    torch.cuda.synchronize()
    for x, y in zip(a[:3], b[:3]):
        x, y = x.float(), y.float()
        assert (x - y).abs().max() <= 2e-2 * y.abs().max()
    for h in range(H):
        r = bo.sla_backward_head(synth.as_f64(q[0, h]), synth.as_f64(k[0, h]), synth.as_f64(v[0, h]),
                                 synth.as_f64(dout[0, h]), mask[0, h], bq, 64, proj_w=synth.as_f64(W), has_bias=True)
        for name, got in (("dQ", a[0]), ("dK", a[1]), ("dV", a[2])):
            _compare(name, got[0, h].float().cpu().numpy(), r[name])


def test_backward_argument_errors():
    dev = torch.device("cuda:0")
    x = torch.zeros((1, 1, 128, 128), dtype=torch.bfloat16, device=dev)
    with pytest.raises(sla.SLAError) as e:
        sla.sla_attention_bwd(x, x, x, x, 128, 64, 0.5, 0.5, phi_kind=3)
    assert e.value.status == sla.ERR_UNSUPPORTED
    with pytest.raises(sla.SLAError) as e:
        sla.sla_attention_bwd(x, x, x, x, 128, 64, 0.5, 0.5, workspace=torch.empty(256, dtype=torch.uint8, device=dev))
    assert e.value.status == sla.ERR_WORKSPACE


def test_projection_gradients_are_deterministic_and_bias_alone_can_be_asked_for():
    """dproj_w and dproj_b are per-workgroup partial sums added in a fixed order: two calls give the same
    bits (a shape with several workgroups per head), and asking for the bias gradient alone gives the same
    bias gradient as asking for both."""
    cfg = synth.custom_config(1, 3, (8, 16, 32), block_q=128, topk_ratio=0.2, marginal_ratio=0.4, use_proj=True, cfg_id=305)
    q, k, v = synth.make_qkv(cfg)
    dout = synth.make_qkv(cfg, seed=5)[2]
    dev = torch.device("cuda:0")
    qd, kd, vd, dd, Wd = (t.to(dev) for t in (q, k, v, dout, synth.make_proj(cfg)))
    run = lambda **kw: sla.sla_attention_bwd(qd, kd, vd, dd, 128, 64, 0.2, 0.4, proj_w=Wd, **kw)
    a = run(want_dw=True, want_db=True)
    b = run(want_dw=True, want_db=True)
    c = run(want_db=True)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    assert c[3] is None and torch.equal(c[4], a[4])
    ref_b = dout.double().sum(dim=(0, 1, 2)).numpy()           # the bias gradient has a closed form
    assert np.abs(a[4].cpu().numpy() - ref_b).max() <= 1e-4 * np.abs(ref_b).max() + 1e-3


@pytest.mark.parametrize("bq,rc,rm", [(128, 0.25, 0.5), (64, 0.75, 0.25)])
def test_training_step_on_token_major_tensors_gives_the_same_bits(bq, rc, rm):
    """sla_attention_fwd_train_strided + sla_attention_bwd_strided on [B,N,H,d] memory (q, k, v packed in one
    [B,N,3,H,d] buffer, gradients written into another): bit-identical to the contiguous calls, which the tests
    above check against the oracle.  Both dK/dV variants (one and two key blocks per workgroup)."""
    cfg = synth.custom_config(2, 2, (5, 10, 20), block_q=bq, topk_ratio=rc, marginal_ratio=rm, use_proj=True, cfg_id=306)
    q, k, v = synth.make_qkv(cfg)
    dout = synth.make_qkv(cfg, seed=13)[2]
    dev = torch.device("cuda:0")
    qd, kd, vd, dd, Wd = (t.to(dev) for t in (q, k, v, dout, synth.make_proj(cfg)))
    out_ref, saved_ref = sla.sla_attention_fwd_train(qd, kd, vd, bq, 64, rc, rm, proj_w=Wd)
    ref = sla.sla_attention_bwd(qd, kd, vd, dd, bq, 64, rc, rm, proj_w=Wd, want_dw=True, want_db=True, saved=saved_ref)
    B, H, N, d = qd.shape
    packed = torch.stack([t.permute(0, 2, 1, 3) for t in (qd, kd, vd)], dim=2).contiguous()      # [B,N,3,H,d]
    qv, kv, vv = (packed[:, :, i].permute(0, 2, 1, 3) for i in range(3))
    dtm = dd.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    out_tm = torch.empty((B, N, H, d), dtype=torch.bfloat16, device=dev).permute(0, 2, 1, 3)
    saved = sla.sla_attention_fwd_train_strided(qv, kv, vv, out_tm, bq, 64, rc, rm, proj_w=Wd)
    assert torch.equal(out_tm, out_ref) and torch.equal(saved, saved_ref)
    grads = torch.full((B, N, 3, H, d), 7.0, dtype=torch.bfloat16, device=dev)
    gq, gk, gv = (grads[:, :, i].permute(0, 2, 1, 3) for i in range(3))
    for sv in (saved, None):                          # from the saved statistics, and recomputing them
        dw, db = sla.sla_attention_bwd_strided(qv, kv, vv, dtm, gq, gk, gv, bq, 64, rc, rm, proj_w=Wd, want_dw=True,
                                               want_db=True, saved=sv)
        torch.cuda.synchronize()
        if sv is None:
            ref = sla.sla_attention_bwd(qd, kd, vd, dd, bq, 64, rc, rm, proj_w=Wd, want_dw=True, want_db=True)
        for got, want in zip((gq, gk, gv, dw, db), ref):
            assert torch.equal(got, want)


def test_saved_state_of_another_problem_poisons_the_gradients():
    """The state a training forward pass saves names its problem; handed to a backward pass with another number of
    critical blocks per row (same sizes, so the byte count matches) every gradient comes out NaN, not plausibly wrong."""
    cfg = synth.custom_config(1, 2, (5, 10, 20), block_q=128, topk_ratio=0.25, marginal_ratio=0.5, cfg_id=330)
    q, k, v = synth.make_qkv(cfg)
    dout = synth.make_qkv(cfg, seed=7)[2]
    W = synth.make_proj(cfg)
    qd, kd, vd, dd, Wd = (t.cuda() for t in (q, k, v, dout, W))
    out, saved = sla.sla_attention_fwd_train(qd, kd, vd, 128, 64, 0.25, 0.5, proj_w=Wd)
    good = sla.sla_attention_bwd(qd, kd, vd, dd, 128, 64, 0.25, 0.5, proj_w=Wd, saved=saved)
    assert all(torch.isfinite(g.float()).all() for g in good[:3])
    bad = sla.sla_attention_bwd(qd, kd, vd, dd, 128, 64, 0.5, 0.5, proj_w=Wd, saved=saved)   # 8 critical blocks, not 4
    assert all(torch.isnan(g.float()).any() for g in bad[:3])
    junk = torch.zeros_like(saved)
    assert torch.isnan(sla.sla_attention_bwd(qd, kd, vd, dd, 128, 64, 0.25, 0.5, proj_w=Wd, saved=junk)[0].float()).any()



@pytest.mark.parametrize("bq", [128, 64])
def test_backward_of_many_heads(bq):
    """Enough query blocks for two tiles of 32 queries per wavefront in the statistics pass (fewer take one), on a
    ragged sequence (N = 1000: 15 key blocks and 40 keys, a query tile that ends inside it): first and last head
    against the oracle."""
    H = 64
    cfg = synth.custom_config(1, H, (5, 10, 20), block_q=bq, topk_ratio=0.25, marginal_ratio=0.5, use_proj=False, cfg_id=310)
    q, k, v = synth.make_qkv(cfg)
    dout = synth.make_qkv(cfg, seed=7)[2]
    qd, kd, vd, dd = (t.cuda() for t in (q, k, v, dout))
    mask = sla.sla_classify_blocks(qd, kd, bq, 64, 0.25, 0.5, want_scores=False)[0].cpu().numpy()
    dq, dk, dv, _, _ = sla.sla_attention_bwd(qd, kd, vd, dd, bq, 64, 0.25, 0.5, want_dw=False, want_db=False)
    for h in (0, H - 1):
        r = bo.sla_backward_head(*(synth.as_f64(t[0, h]) for t in (q, k, v, dout)), mask[0, h], bq, 64)
        for name, got in (("dQ", dq), ("dK", dk), ("dV", dv)):
            _compare("%s head %d" % (name, h), got[0, h].float().cpu().numpy(), r[name])


@pytest.mark.parametrize("H,grid,bq,rc,rm", [
    (2, (5, 10, 20), 128, 0.25, 0.5),     # one tile of 32 queries per wavefront, a ragged last block
    (2, (5, 10, 20), 64, 0.25, 0.5),
    (64, (5, 10, 20), 128, 0.25, 0.5),    # two of them
    (64, (5, 10, 20), 64, 0.25, 0.5),
    (2, (4, 16, 16), 128, 0.75, 0.25),    # whole blocks; two key blocks per workgroup in dK / dV
])
def test_contiguous_tensors_may_start_at_any_element(H, grid, bq, rc, rm):
    """The calls without strides take contiguous tensors wherever they start (a slice of a flat buffer): the kernels that
    copy rows of 16-byte units straight to LDS take others through registers.  Same values, so the same bits."""
    cfg = synth.custom_config(1, H, grid, block_q=bq, topk_ratio=rc, marginal_ratio=rm, use_proj=True, cfg_id=340)
    q, k, v = synth.make_qkv(cfg)
    even = [t.cuda() for t in (q, k, v, synth.make_qkv(cfg, seed=7)[2], synth.make_proj(cfg))]

    def moved(t, elements):
        flat = torch.zeros(t.numel() + 8, dtype=t.dtype, device="cuda")
        view = flat[elements:elements + t.numel()].view(t.shape)
        view.copy_(t)
        assert view.is_contiguous() and view.data_ptr() % 16 == 2 * elements
        return view
    for shift in (1, 4):
        odd = [moved(t, shift) for t in even]
        got_out, got_saved = sla.sla_attention_fwd_train(*odd[:3], bq, 64, rc, rm, proj_w=odd[4])
        out, saved = sla.sla_attention_fwd_train(*even[:3], bq, 64, rc, rm, proj_w=even[4])
        assert torch.equal(got_out, out) and torch.equal(got_saved, saved)
        for state in (None, saved):
            kw = dict(want_dw=True, want_db=True, saved=state)
            grads = tuple(moved(torch.zeros_like(t), shift) for t in even[:3])
            want = sla.sla_attention_bwd(*even[:4], bq, 64, rc, rm, proj_w=even[4], **kw)
            got = sla.sla_attention_bwd(*odd[:4], bq, 64, rc, rm, proj_w=odd[4], grads=grads, **kw)
            for name, a, b in zip(("dQ", "dK", "dV", "dW", "db"), got, want):
                assert torch.equal(a, b), (name, shift, state is None)


@pytest.mark.parametrize("H,N,bq", [(4, 4617, 64), (12, 32760, 128), (40, 8000, 64)])
def test_bias_gradient_is_summed_without_long_chains(H, N, bq):
    """db = sum of dout over every token, in fp32.  An addition rounds its result by a relative variance of about
    0.18 u^2 (u = 2^-24, mantissas spread evenly over a binade); of sums of random signs a chain of m equal additions
    then costs m / 2 of those, a pairwise sum 1 + 1/2 + 1/4 + ...  The order asked for: a workgroup's query blocks one
    after the other (256 workgroups; a block's own tokens add up all but exactly), its partials by 16 threads in four
    chains of four that are joined pairwise, the 16 pairwise.  Root mean square over four draws, a tenth allowed."""
    squares = []
    for seed in range(4):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        x = [torch.randn((1, H, N, 128), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4)]
        db = sla.sla_attention_bwd(*x, bq, 64, 0.05, 0.3, want_db=True)[4].double()
        ref = x[3].double().sum((0, 1, 2))
        squares.append(float(((db - ref).norm() / ref.norm()) ** 2))
    err = np.mean(squares) ** 0.5
    blocks = H * -(-N // bq) / 256
    bound = 1.1 * 2.0 ** -24 * (0.18 * (blocks / 2 + 4 / 2 + 1.5 + 1.875)) ** 0.5
    print("db %d heads x %d: %.2e (bound %.2e)" % (H, N, err, bound))
    assert err <= bound


def _token_major(t):
    return t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)


@pytest.mark.parametrize("bq", [128, 64])
def test_training_step_of_many_heads_on_token_major_tensors_gives_the_same_bits(bq):
    """Enough query blocks for two tiles of 32 queries per wavefront, on [B,N,H,d] memory: the statistics and dQ kernels'
    instances for strided tensors against those for contiguous ones (which test_backward_of_many_heads checks against
    the oracle), from the saved state and without it, on a ragged sequence."""
    cfg = synth.custom_config(1, 64, (5, 10, 20), block_q=bq, topk_ratio=0.25, marginal_ratio=0.5, use_proj=True, cfg_id=311)
    q, k, v = (t.cuda() for t in synth.make_qkv(cfg))
    dout, W = synth.make_qkv(cfg, seed=7)[2].cuda(), synth.make_proj(cfg).cuda()
    out, saved = sla.sla_attention_fwd_train(q, k, v, bq, 64, 0.25, 0.5, proj_w=W)
    tm = [_token_major(t) for t in (q, k, v, dout)]
    grads = [torch.full_like(t, 7.0) for t in tm[:3]]
    assert not grads[0].is_contiguous()
    for state in (saved, None):
        kw = dict(proj_w=W, want_dw=True, want_db=True, saved=state)
        ref = sla.sla_attention_bwd(q, k, v, dout, bq, 64, 0.25, 0.5, **kw)
        dw, db = sla.sla_attention_bwd_strided(*tm, *grads, bq, 64, 0.25, 0.5, **kw)
        for name, got, want in zip(("dQ", "dK", "dV", "dW", "db"), (*grads, dw, db), ref):
            assert torch.equal(got, want), (name, state is None)


@pytest.mark.parametrize("grid,bq,H", [((1, 5, 5), 64, 1024), ((1, 5, 5), 128, 512), ((1, 9, 9), 64, 512), ((1, 9, 9), 128, 512)])
def test_backward_of_many_short_sequences(grid, bq, H):
    """One or two key blocks, the last one ragged (25 keys; 17), two query tiles per wavefront: the copy rings at their
    shortest, with missing keys in the first block of the walk.  First and last head against the oracle, in both layouts."""
    cfg = synth.custom_config(1, H, grid, block_q=bq, topk_ratio=0.5, marginal_ratio=0.5, use_proj=False, cfg_id=312)
    q, k, v = synth.make_qkv(cfg)
    dout = synth.make_qkv(cfg, seed=7)[2]
    dev = [t.cuda() for t in (q, k, v, dout)]
    mask = sla.sla_classify_blocks(dev[0], dev[1], bq, 64, 0.5, 0.5, want_scores=False)[0].cpu().numpy()
    got = sla.sla_attention_bwd(*dev, bq, 64, 0.5, 0.5)[:3]
    for h in (0, H - 1):
        r = bo.sla_backward_head(*(synth.as_f64(t[0, h]) for t in (q, k, v, dout)), mask[0, h], bq, 64)
        for name, g in zip(("dQ", "dK", "dV"), got):
            _compare("%s head %d" % (name, h), g[0, h].float().cpu().numpy(), r[name])
    grads = [torch.full_like(_token_major(t), 7.0) for t in dev[:3]]
    sla.sla_attention_bwd_strided(*(_token_major(t) for t in dev), *grads, bq, 64, 0.5, 0.5)
    assert all(torch.equal(a, b) for a, b in zip(grads, got))


@pytest.mark.parametrize("token_bytes", [(1 << 26) - 16, 1 << 26])
def test_backward_at_token_strides_the_offsets_just_reach_and_no_longer_reach(token_bytes):
    """q, k, v and dout as columns of one buffer whose rows lie 64 MiB apart: the largest stride at which a lane's offset
    into a tile fits 32 bits, and the next one, which takes addresses per lane.  The contiguous call's bits, for one and
    two query tiles per wavefront (the second: 512 heads, 97 tokens in two key blocks); so for the 16-bit forward pass,
    in steps of one key tile and of two, on the values and on INT8 codes of Q and K (V alone is the caller's there)."""
    N, token = 97, token_bytes // 2
    buf = torch.empty(N * token, dtype=torch.bfloat16, device="cuda")      # (6 GB, of which 97 rows of 0.5 MB are used)
    for H, bq in ((2, 64), (2, 128), (512, 128), (512, 64)):
        cfg = synth.custom_config(1, H, (1, 1, N), block_q=bq, topk_ratio=0.5, marginal_ratio=0.5, use_proj=False, cfg_id=313)
        dev = [t.cuda() for t in (*synth.make_qkv(cfg), synth.make_qkv(cfg, seed=7)[2])]
        far = []
        for i, t in enumerate(dev):
            view = buf.as_strided((1, H, N, 128), (N * token, 128, token, 1), i * H * 128)
            view.copy_(t)
            far.append(view)
        want = sla.sla_attention_bwd(*dev, bq, 64, 0.5, 0.5)[:3]
        grads = [torch.full_like(t, 7.0) for t in dev[:3]]
        sla.sla_attention_bwd_strided(*far, *grads, bq, 64, 0.5, 0.5)
        for name, a, b in zip(("dQ", "dK", "dV"), grads, want):
            assert torch.equal(a, b), (name, H, bq)
        for mode in (sla.QUANT_NONE, sla.QUANT_QK_INT8):
            want = sla.sla_attention_fwd(*dev[:3], bq, 64, 0.5, 0.5, quant_mode=mode)
            out = torch.full_like(want, 7.0)
            sla.sla_attention_fwd_strided(*far[:3], out, bq, 64, 0.5, 0.5, quant_mode=mode,
                                          workspace=sla.alloc_workspace(1, H, N, 128, bq, 64, 0.5, 0.5, quant_mode=mode))
            assert torch.equal(out, want), (mode, H, bq)
