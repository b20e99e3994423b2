"""GPU parity of the W8A8 Linear layer (through the C ABI) against the CPU oracle:
the quantiser's codes and scales, the INT8 product with its block-scale accumulation
given those codes, and the whole layer from bf16 inputs."""
import numpy as np
import pytest
import torch

from oracle import w8a8_oracle as wo
from paper_2512_16093_amd import binding as sla
from paper_2512_16093_amd import synth

pytestmark = pytest.mark.gpu

# (M, K, N): one token; ragged token tails; one and many feature blocks; several output tiles
SHAPES = [(1, 128, 128), (300, 384, 256), (257, 256, 128), (1000, 1024, 512), (640, 2048, 384)]


def check_codes(gpu_codes, gpu_scales, A, what):
    codes, scales = wo.quantize_blockwise(A)
    # scales: max|block| / 127 evaluated in fp32 on the GPU, in fp64 here
    assert np.allclose(gpu_scales, scales, rtol=3e-7, atol=0), what
    # codes: the correctly rounded quotient 127 x / amax on both sides, exact ties to the even code: identical
    assert np.array_equal(gpu_codes.astype(np.float64), codes), (what, int((gpu_codes != codes).sum()))


def product_tolerance(ref, sX, sW, K):
    """bf16 rounding of the result (relative 2^-9, doubled) plus the fp32 accumulation of the block
    sums.  The kernel adds each block sum together with a constant of about 2^23.4 integer steps
    (it reads the integer accumulator as a float, see the kernel's header) and removes the
    constants every fourth block, so a running sum stays below 2^26 steps and every fma rounds by
    at most 2 steps s_X s_W: at most 2 K / 128 steps in all (a worst case; the errors are random)."""
    return 2.0 ** -8 * np.abs(ref) + (2.0 * K / 128 + 1.0) * sX.max() * sW.max()


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_quantiser_matches_oracle(M, K, N):
    x, w, _ = synth.make_linear_inputs(M, K, N)
    ws = sla.w8a8_quantize_act(x.cuda())
    xc, xs = sla.w8a8_debug_unpack(ws, False, M, K)
    check_codes(xc.cpu().numpy(), xs.cpu().numpy(), synth.as_f64(x), "activations %s" % ((M, K),))
    wq = sla.w8a8_quantize_weight(w.cuda())
    wc, wsc = sla.w8a8_debug_unpack(wq, True, N, K)
    check_codes(wc.cpu().numpy(), wsc.cpu().numpy(), synth.as_f64(w), "weights %s" % ((N, K),))


@pytest.mark.parametrize("M,K,N", SHAPES)
@pytest.mark.parametrize("with_bias", [True, False])
def test_product_matches_oracle_on_the_same_codes(M, K, N, with_bias):
    x, w, b = synth.make_linear_inputs(M, K, N, seed=1, with_bias=with_bias)
    xd, wd = x.cuda(), w.cuda()
    bd = None if b is None else b.cuda()
    wq = sla.w8a8_quantize_weight(wd)
    ws = sla.w8a8_quantize_act(xd)
    y = sla.w8a8_gemm_fwd(ws, wq, M, N, K, bias=bd).float().cpu().numpy()
    xc, xs = (t.cpu().numpy().astype(np.float64) for t in sla.w8a8_debug_unpack(ws, False, M, K))
    wc, wsc = (t.cpu().numpy().astype(np.float64) for t in sla.w8a8_debug_unpack(wq, True, N, K))
    ref = wo.linear_from_codes(xc, xs, wc, wsc, None if b is None else synth.as_f64(b))
    assert np.all(np.abs(y - ref) <= product_tolerance(ref, xs, wsc, K)), np.abs(y - ref).max()


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_whole_layer_matches_oracle(M, K, N):
    x, w, b = synth.make_linear_inputs(M, K, N, seed=2)
    wq = sla.w8a8_quantize_weight(w.cuda())
    y = sla.w8a8_linear_fwd(x.cuda(), wq, N, bias=b.cuda()).float().cpu().numpy()
    ref, parts = wo.w8a8_linear(synth.as_f64(x), synth.as_f64(w), synth.as_f64(b))
    # (the codes are the oracle's, see test_quantiser_matches_oracle: only the product's own tolerance applies)
    tol = product_tolerance(ref, parts["sX"], parts["sW"], K)
    assert np.all(np.abs(y - ref) <= tol), np.abs(y - ref).max()
    assert np.linalg.norm(y - ref) / np.linalg.norm(ref) < 3e-3
    # and the layer does its job: close to the unquantised product (a block's scale follows its
    # outlier features, so the other features of the block keep only a few bits: several percent)
    dense = synth.as_f64(x) @ synth.as_f64(w).T + synth.as_f64(b)
    assert np.linalg.norm(y - dense) / np.linalg.norm(dense) < 0.15


def test_exactly_representable_inputs_lose_only_the_accumulation_steps():
    """Integer codes times power-of-two scales, every block holding a 127: quantisation is lossless,
    so the only errors left are the accumulation's (at most 2 steps s_X s_W = 1/8 per block, two
    blocks here) and the bf16 rounding of the output."""
    g = np.random.default_rng(3)
    M, K, N = 300, 256, 256
    Xi = g.integers(-3, 4, size=(M, K)).astype(np.float32)
    Wi = g.integers(-2, 3, size=(N, K)).astype(np.float32)
    Xi[::128, ::128] = 127.0
    Wi[::128, ::128] = 127.0
    Xi[::128, 1::128] = 0.0
    x = torch.from_numpy(Xi * 0.25).to(torch.bfloat16)
    w = torch.from_numpy(Wi * 0.5).to(torch.bfloat16)
    xd, wd = x.cuda(), w.cuda()
    wq = sla.w8a8_quantize_weight(wd)
    ws = sla.w8a8_quantize_act(xd)
    xc, xs = sla.w8a8_debug_unpack(ws, False, M, K)
    wc, wsc = sla.w8a8_debug_unpack(wq, True, N, K)
    assert np.array_equal(xc.cpu().numpy(), Xi) and np.array_equal(wc.cpu().numpy(), Wi)      # lossless codes
    assert (xs == 0.25).all() and (wsc == 0.5).all()
    y = sla.w8a8_linear_fwd(xd, wq, N).float().cpu().numpy()
    ref = (Xi * 0.25).astype(np.float64) @ (Wi * 0.5).astype(np.float64).T
    assert np.all(np.abs(y - ref) <= 4 * 0.125 + 2.0 ** -9 * np.abs(ref))
    assert (y == ref).mean() > 0.5          # and most results are exact


def test_deterministic_and_workspace_reuse():
    x, w, b = synth.make_linear_inputs(500, 512, 256, seed=4)
    xd, bd = x.cuda(), b.cuda()
    wq = sla.w8a8_quantize_weight(w.cuda())
    ws = sla.w8a8_alloc_workspace(500, 512)
    y1 = sla.w8a8_linear_fwd(xd, wq, 256, bias=bd, workspace=ws).clone()
    sla.w8a8_linear_fwd(xd[:100].contiguous(), wq, 256, bias=bd, workspace=ws)   # a smaller call in between
    y2 = sla.w8a8_linear_fwd(xd, wq, 256, bias=bd, workspace=ws)
    assert torch.equal(y1, y2)
    assert torch.equal(x, xd.cpu())


def test_long_contraction_feed_forward_down_shape():
    """K = 13824 (108 feature blocks, the feed-forward down projection of a Wan-14B block): the
    longest accumulation of block sums the layer sees, on 1000 tokens."""
    M, K, N = 1000, 13824, 5120
    x, w, b = synth.make_linear_inputs(M, K, N, seed=5)
    wq = sla.w8a8_quantize_weight(w.cuda())
    ws = sla.w8a8_quantize_act(x.cuda())
    y = sla.w8a8_gemm_fwd(ws, wq, M, N, K, bias=b.cuda()).float().cpu().numpy()
    xc, xs = (t.cpu().numpy().astype(np.float64) for t in sla.w8a8_debug_unpack(ws, False, M, K))
    wc, wsc = (t.cpu().numpy().astype(np.float64) for t in sla.w8a8_debug_unpack(wq, True, N, K))
    ref = wo.linear_from_codes(xc, xs, wc, wsc, synth.as_f64(b))
    err = np.abs(y - ref)
    assert np.all(err <= product_tolerance(ref, xs, wsc, K)), err.max()
    # what the accumulation adds on top of the bf16 rounding of the output: in steps of the largest
    # block it stays inside the worst-case bound, and as a relative error it is smaller than the
    # output rounding itself (both are ~100x below the rounding of the INT8 codes)
    excess = (err - 2.0 ** -9 * np.abs(ref)).max() / (xs.max() * wsc.max())
    rel = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    print("w8a8 K=13824: accumulation error beyond output rounding: %.1f steps (bound %d); relative error %.2e"
          % (max(excess, 0.0), 2 * K // 128 + 1, rel))
    assert rel < 3e-3


def test_full_size_attention_projection_sampled():
    """The layer at the size the benchmark times (75600 tokens, 5120 -> 5120): the oracle on whole
    quantisation row blocks -- the first, one in the middle and the ragged last one (75600 =
    590 * 128 + 80) -- against all output features."""
    M, K, N = 75600, 5120, 5120
    x, w, b = synth.make_linear_inputs(M, K, N)
    print("running the GPU layer", flush=True)
    wq = sla.w8a8_quantize_weight(w.cuda())
    y = sla.w8a8_linear_fwd(x.cuda(), wq, N, bias=b.cuda())
    torch.cuda.synchronize()
    assert torch.isfinite(y.float()).all()
    print("oracle: quantising the weight", flush=True)
    W8, sW = wo.quantize_blockwise(synth.as_f64(w))
    worst = 0.0
    for rb in (0, 295, 590):
        rows = slice(rb * 128, min((rb + 1) * 128, M))
        print("oracle on token block", rb, flush=True)
        X8, sX = wo.quantize_blockwise(synth.as_f64(x[rows]))
        ref = wo.linear_from_codes(X8, sX, W8, sW, synth.as_f64(b))
        got = y[rows].float().cpu().numpy()
        tol = product_tolerance(ref, sX, sW, K) + 127.0 * 4 * sX.max() * sW.max()
        assert np.all(np.abs(got - ref) <= tol), (rb, np.abs(got - ref).max())
        rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        assert rel < 3e-3, (rb, rel)
        worst = max(worst, rel)
    print("w8a8 75600 x 5120 -> 5120: worst relative error of a sampled token block %.2e" % worst)


@pytest.mark.parametrize("M,K,N", [
    (1, 256, 128), (33, 640, 384),           # fewer feature blocks than wavefronts that split them; 32-row tiles, one row over
    (31, 1024, 8192), (32, 256, 5120),       # 32 x 32 tiles, contraction split four and eight ways
    (65, 384, 8192), (129, 4352, 5120),      # 32 x 64 tiles split four ways; 64 x 64 split eight ways (34 blocks, uneven runs)
    (200, 384, 8192), (257, 640, 8192),      # 32 x 64 and 64 x 64 split in two
    (1023, 384, 4096), (1025, 256, 5120),    # 64 x 64, not split; two feature blocks
    (2049, 384, 3712),                       # the large tiles: nine bands of token tiles, a ragged last patch
    # long contractions in one round of wide tiles; by four wavefronts 64 x 96 (the last tile of a row reaches past the outputs,
    # the last of a column holds one row of tokens), the same with an odd number of blocks, 64 x 128, 64 x 160 and 128 x 96
    (1025, 2048, 1024), (1090, 4224, 1152), (200, 2048, 8064), (1200, 2048, 1792), (2050, 2048, 1408),
    (257, 2048, 12288), (833, 3968, 5120), (3000, 3968, 1920),   # by two: 64 x 128, 64 x 160, 128 x 96
])
def test_every_tile_and_split_of_the_product(M, K, N):
    """The product's variants (tile size, ways the contraction is split) at the edges of what selects them, against
    the oracle on the same codes, with the tolerance of the other product tests."""
    x, w, b = synth.make_linear_inputs(M, K, N, seed=6)
    wq = sla.w8a8_quantize_weight(w.cuda())
    ws = sla.w8a8_quantize_act(x.cuda())
    guard = torch.full((M + 64, N), 7.0, dtype=torch.bfloat16, device="cuda")   # rows past M must stay as they are
    y = sla.w8a8_gemm_fwd(ws, wq, M, N, K, bias=b.cuda(), out=guard[:M]).float().cpu().numpy()
    assert (guard[M:] == 7.0).all()
    xc, xs = (t.cpu().numpy().astype(np.float64) for t in sla.w8a8_debug_unpack(ws, False, M, K))
    wc, wsc = (t.cpu().numpy().astype(np.float64) for t in sla.w8a8_debug_unpack(wq, True, N, K))
    ref = wo.linear_from_codes(xc, xs, wc, wsc, synth.as_f64(b))
    assert np.all(np.abs(y - ref) <= product_tolerance(ref, xs, wsc, K)), np.abs(y - ref).max()


@pytest.mark.parametrize("M,K,N", [
    (33, 640, 384), (5, 1152, 2048),          # one block to a wavefront (eight ways); runs of one and two blocks
    (200, 384, 8192), (513, 640, 5120),       # two ways: runs of one and two, of two and three blocks
    (128, 1664, 5120), (512, 5120, 1024),     # eight ways over 13 blocks, four over 40
    (1500, 128, 5120),                        # one block in all
])
def test_split_contraction_is_no_less_precise_than_one_walk(M, K, N):
    """Splitting the contraction must not cost precision.  The yardstick is the kernel's arithmetic in ONE walk over the
    feature blocks, formed here on the same codes: per block one fma of (constant +- block sum) in fp32, constants of
    alternating sign, their sum (a rounded product) taken out at the end.  Counted is how many outputs are not the correctly rounded bf16 of
    the exact sum; both counts are of M x N outputs, their own scatter is well under the 2 % (and 50) allowed."""
    missed, allowed = _not_the_rounded_exact_sum(M, K, N, 9)
    print("w8a8 %d x %d -> %d: %d outputs not the rounded exact sum, one walk %d" % (M, K, N, missed, allowed))
    assert missed <= 1.02 * allowed + 50


@pytest.mark.parametrize("M,K,N", [
    (512, 5120, 5120), (1090, 4224, 1152),    # by four wavefronts: 40 blocks, 33 (the last run's last does not exist)
    (2050, 2048, 1408), (833, 3968, 5120),    # 128 x 96 by four, 64 x 160 by two (31 blocks)
])
def test_wide_tiles_are_no_less_precise_than_one_walk(M, K, N):
    """The same of the wide tiles, whose runs all have an even number of blocks.  Which constants are left standing while a run
    goes on depends on where the blocks with outlier features (scales ten to thirty times the others') lie in it: the ratio of
    the two counts was 0.46 to 1.31 over twelve inputs of these sizes, 0.75 to 0.89 on average, so eight inputs are added up
    (their mean scatters by a third of the single ones' 0.2)."""
    missed, allowed = np.sum([_not_the_rounded_exact_sum(M, K, N, seed) for seed in range(9, 17)], axis=0)
    print("w8a8 %d x %d -> %d: %d outputs not the rounded exact sum, one walk %d" % (M, K, N, missed, allowed))
    assert missed <= allowed


def _not_the_rounded_exact_sum(M, K, N, seed):
    """(outputs of the product, outputs of one walk) that are not the exact sum rounded to bf16."""
    x, w, _ = synth.make_linear_inputs(M, K, N, seed=seed)
    wq = sla.w8a8_quantize_weight(w.cuda())
    ws = sla.w8a8_quantize_act(x.cuda())
    y = sla.w8a8_gemm_fwd(ws, wq, M, N, K)
    (xc, xs), (wc, wsc) = sla.w8a8_debug_unpack(ws, False, M, K), sla.w8a8_debug_unpack(wq, True, N, K)
    rows = lambda s, n: s.repeat_interleave(128, 0)[:n]
    c0 = np.int32(0x3E22F983).view(np.float32).item()
    exact = torch.zeros((M, N), dtype=torch.float64, device="cuda")
    walk, csum = torch.zeros((M, N), dtype=torch.float32, device="cuda"), torch.zeros((M, N), dtype=torch.float32, device="cuda")
    for kb in range(K // 128):
        block = xc[:, 128 * kb:128 * kb + 128].double() @ wc[:, 128 * kb:128 * kb + 128].double().t().contiguous()
        scale = rows(xs[:, kb:kb + 1], M) * rows(wsc[:, kb:kb + 1], N).t()          # fp32, as the kernel forms it
        exact += block * (rows(xs[:, kb:kb + 1], M).double() * rows(wsc[:, kb:kb + 1], N).double().t())
        sc = (scale * 2.0 ** 26 * (-1.0) ** kb).double()
        acc = c0 + block * 2.0 ** -26 * (-1.0) ** kb                                # exact: a float of the binade [1/8, 1/4)
        walk = (acc * sc + walk.double()).float()                                   # (one rounding to fp32, as in an fma)
        csum = (csum.double() + sc).float()
    walk = walk - c0 * csum
    rounded = exact.to(torch.bfloat16)
    return int((y != rounded).sum()), int((walk.to(torch.bfloat16) != rounded).sum())


@pytest.mark.parametrize("M,K,N", [
    (200, 640, 128), (129, 256, 128),         # one column of output tiles; more tokens than outputs by one
    (2000, 384, 256), (5000, 1280, 384),      # several, not split and split two ways, ragged last tokens
    (257, 128, 256), (256, 128, 256),         # one more token than outputs; as many
])
def test_small_tiles_of_more_tokens_than_outputs(M, K, N):
    """The small tiles are dealt to the XCDs along the smaller operand: every tile is still there, once, against the
    oracle on the same codes with the tolerance of the other product tests."""
    x, w, b = synth.make_linear_inputs(M, K, N, seed=8)
    wq = sla.w8a8_quantize_weight(w.cuda())
    ws = sla.w8a8_quantize_act(x.cuda())
    guard = torch.full((M + 64, N), 7.0, dtype=torch.bfloat16, device="cuda")   # rows past M must stay as they are
    y = sla.w8a8_gemm_fwd(ws, wq, M, N, K, bias=b.cuda(), out=guard[:M]).float().cpu().numpy()
    assert (guard[M:] == 7.0).all()
    xc, xs = (t.cpu().numpy().astype(np.float64) for t in sla.w8a8_debug_unpack(ws, False, M, K))
    wc, wsc = (t.cpu().numpy().astype(np.float64) for t in sla.w8a8_debug_unpack(wq, True, N, K))
    ref = wo.linear_from_codes(xc, xs, wc, wsc, synth.as_f64(b))
    assert np.all(np.abs(y - ref) <= product_tolerance(ref, xs, wsc, K)), np.abs(y - ref).max()
