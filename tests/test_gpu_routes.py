"""Calls whose launches depend on the problem's size: the same slice, taken by either route, must give the same bits."""
import pytest
import torch

from paper_2512_16093_amd import binding as sla

pytestmark = pytest.mark.gpu

D = 128


def _qkv(H, N, seed=3):
    g = torch.Generator(device="cuda").manual_seed(seed)
    xs = [torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3)]
    xs[1] += 2.0 * torch.randn((D,), generator=g, device="cuda", dtype=torch.bfloat16)
    return xs


def _weight(offset, seed=4):
    g = torch.Generator(device="cuda").manual_seed(seed)
    buf = (torch.randn((D * D + offset,), generator=g, device="cuda") / D ** 0.5).to(torch.bfloat16)
    return buf[offset:].view(D, D)


@pytest.mark.parametrize("quant", [sla.QUANT_QK_INT8_PV_FP8, sla.QUANT_NONE])
@pytest.mark.parametrize("N, block_q, rc, rm, w", [
    (25, 64, 1.0, 0.0, None),     # one short key block, no linear branch (in 16 bits both sides take the same launches)
    (81, 128, 0.5, 0.5, 0),       # two key blocks, the projection aligned
    (189, 64, 0.34, 0.66, 1),     # three query blocks (one wavefront of the four without a row), W off by two bytes
    (1000, 128, 0.2, 0.4, None),  # a ragged last key block, no projection
    (4033, 64, 0.1, 0.2, 1),      # 64 key blocks, the last of one token: the longest slice of the one-launch route
    (4097, 128, 0.1, 0.2, 0),     # 65: the shortest of the other, whatever its company: both sides take the same launches
])
def test_few_and_many_slices_give_the_same_bits(N, block_q, rc, rm, w, quant):
    """Few slices of few blocks are classified, joined and quantised in one launch, many of them in two; a slice's
    result does not depend on its company."""
    groups = ((N + block_q - 1) // block_q + 3) // 4
    many = 1024 // groups + 1
    q, k, v = _qkv(many, N)
    kw = dict(proj_w=None if w is None else _weight(w), quant_mode=quant)
    whole = sla.sla_attention_fwd(q, k, v, block_q, 64, rc, rm, **kw)
    pick = [0, many // 2, many - 1]
    few = sla.sla_attention_fwd(*(x[:, pick].contiguous() for x in (q, k, v)), block_q, 64, rc, rm, **kw)
    assert torch.isfinite(few).all()
    assert torch.equal(whole[:, pick], few)


@pytest.mark.parametrize("saved", [True, False])
@pytest.mark.parametrize("N, block_q, rc, rm, w, phi", [
    (81, 128, 0.5, 0.5, 0, sla.PHI_ELU1),        # two key blocks, one query block
    (189, 64, 0.34, 0.66, None, sla.PHI_RELU),   # three query blocks, no projection
    (1000, 64, 0.2, 0.4, 1, sla.PHI_SOFTMAX),    # a ragged last block, W off by two bytes
    (4033, 128, 0.1, 0.2, 0, sla.PHI_ELU1),      # 64 key blocks, the last of one token
])
def test_gradients_of_few_and_many_slices_have_the_same_bits(N, block_q, rc, rm, w, phi, saved):
    """The backward pass takes more from the launch that few slices share: the mask, the unprojected summaries, delta."""
    many = 1024 // (((N + block_q - 1) // block_q + 3) // 4) + 1
    q, k, v = _qkv(many, N)
    do = _qkv(many, N, seed=5)[2]
    kw = dict(proj_w=None if w is None else _weight(w), phi_kind=phi)

    def grads(*xs):
        state = sla.sla_attention_fwd_train(*xs[:3], block_q, 64, rc, rm, **kw)[1] if saved else None
        return sla.sla_attention_bwd(*xs, block_q, 64, rc, rm, saved=state, **kw)[:3]

    whole = grads(q, k, v, do)
    pick = [0, many // 2, many - 1]
    few = grads(*(x[:, pick].contiguous() for x in (q, k, v, do)))
    for a, b in zip(whole, few):
        assert torch.isfinite(b).all()
        assert torch.equal(a[:, pick], b)


@pytest.mark.parametrize("M, K, N", [
    (2032, 256, 2048),    # 128 tiles of 256 x 128 (the last token tile ragged), two feature blocks: large tiles
    (1792, 256, 2304),    # 126: small ones
    (2300, 384, 2304),    # 162 tiles, three blocks: large
    (2560, 640, 2048),    # 160 tiles, five blocks: large
    (2300, 640, 2176),    # 153: small
    (6145, 128, 1024),    # one feature block, 25 token tiles of which the last holds one token
    (2560, 768, 2560),    # 200 tiles, six blocks: large
    (2304, 768, 2816),    # 198: small
    (129, 2560, 8960),    # one round of 64 x 128 tiles, of whose rows of 32 tokens one in six does not exist: 32 x 64 instead
    (2290, 2176, 1280),   # 17 blocks dealt as 4, 4, 4 and 5 to the wavefronts of 128 x 96 tiles: small
    (140, 4096, 5376),    # 252 tiles of 64 x 64, one round of eight wavefronts each
    (80, 4096, 8832),     # 276, more than one round: wide ones
])
@pytest.mark.parametrize("with_bias", [True, False])
def test_linear_layer_on_both_sides_of_the_tile_rule(M, K, N, with_bias):
    """Against the product of the layer's own codes in 64 bits.  Bound per output: a bf16 step (twice its rounding), and of each of
    the K / 128 blocks two steps of its scale (the accumulation rounds at a magnitude of at most 2^25 steps)."""
    g = torch.Generator(device="cuda").manual_seed(M + K)
    x = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((N, K), generator=g, device="cuda") / K ** 0.5).to(torch.bfloat16)
    b = (0.1 * torch.randn((N,), generator=g, device="cuda")).to(torch.bfloat16) if with_bias else None
    wq = sla.w8a8_quantize_weight(w)
    xc, xs = sla.w8a8_debug_unpack(sla.w8a8_quantize_act(x), False, M, K)
    wc, ws = sla.w8a8_debug_unpack(wq, True, N, K)
    ref = torch.zeros((M, N), dtype=torch.float64, device="cuda") + (b.double() if with_bias else 0.0)
    steps = torch.zeros((M, N), dtype=torch.float64, device="cuda")
    for kb in range(K // 128):
        scale = xs[:, kb].double().repeat_interleave(128)[:M, None] * ws[:, kb].double().repeat_interleave(128)[None, :]
        ref += scale * (xc[:, kb * 128:(kb + 1) * 128].double() @ wc[:, kb * 128:(kb + 1) * 128].double().T)
        steps += 2.0 * scale
    y = sla.w8a8_linear_fwd(x, wq, N, bias=b).double()
    assert ((y - ref).abs() <= steps + 2.0 ** -8 * ref.abs()).all()
    assert torch.linalg.norm(y - ref) / torch.linalg.norm(ref) < 3e-3


@pytest.mark.parametrize("with_bias", [True, False])
@pytest.mark.parametrize("M, K, N", [
    (1025, 2048, 1024),   # 64 x 96: the last tile of a row reaches 32 outputs past the end, one token in the last row of tiles
    (1090, 4224, 1152),   # the same with 33 feature blocks: the last wavefront has one that does not exist
    (200, 2048, 8064),    # 64 x 128
    (1200, 2048, 1792),   # 64 x 160, the last tile of a row reaches 128 outputs past the end
    (2050, 2048, 1408),   # 128 x 96
    (257, 2048, 12288),   # 64 x 128 by two wavefronts
    (833, 3968, 5120),    # 64 x 160 by two, 31 blocks
    (3000, 3968, 1920),   # 128 x 96 by two
    (65, 2048, 16384),    # the fewest tokens
])
def test_linear_layer_in_wide_tiles(M, K, N, with_bias):
    """Middling sizes with long contractions; the bound is that of the test above."""
    test_linear_layer_on_both_sides_of_the_tile_rule(M, K, N, with_bias)


@pytest.mark.parametrize("Tq, block_q", [(1, 128), (7, 64), (8, 128), (23, 128), (24, 64), (32, 64), (33, 64), (33, 128), (40, 128), (41, 128),
                                          (48, 64), (49, 64)])
def test_sums_of_short_heads_and_of_long_ones_have_the_same_bits(Tq, block_q):
    """Heads of up to 80 key blocks and 48 query blocks go from memory to registers, others are staged: the same blocks in
    front of more tokens whose key blocks nobody holds as marginal give the same rows."""
    H, N, longer = 3, Tq * block_q - 5, 87 * 64 + 9
    q, k, v = _qkv(H, longer)
    g = torch.Generator(device="cuda").manual_seed(Tq)
    Tk, whole = N // 64, (longer + 63) // 64        # (of the short head's last, ragged key block nothing is marginal)
    mask = torch.full((1, H, (longer + block_q - 1) // block_q, whole), -1, dtype=torch.int8, device="cuda")
    mask[:, :, :Tq, :Tk] = torch.randint(-1, 2, (1, H, Tq, Tk), generator=g, device="cuda", dtype=torch.int8)
    short = [x[:, :, :N].contiguous() for x in (q, k, v)]
    few = sla.sla_linear_attn_fwd(*short, mask[:, :, :Tq, :(N + 63) // 64].contiguous(), block_q, 64, proj_w=_weight(0))
    more = sla.sla_linear_attn_fwd(q, k, v, mask, block_q, 64, proj_w=_weight(0))
    assert torch.isfinite(few).all()
    assert Tk == 1 or few.abs().max() > 0
    assert torch.equal(few, more[:, :, :N])


@pytest.mark.parametrize("H, N, block_q, rc, rm", [
    (9, 4033, 128, 0.1, 0.2),    # 9 x 64 key blocks: just more than the chip holds at a time, all in the order of their lists' lengths
    (41, 1000, 64, 0.2, 0.4),    # 41 x 16, a last group of eight that is short
    (513, 65, 64, 0.5, 0.0),     # two query blocks per slice: no room for an order, the order of the key blocks
    (60, 8192, 128, 0.05, 0.1),  # Q and dO of the last 56 heads fit the memory-side cache: four heads before them in their own order
])
def test_order_of_the_key_blocks_leaves_their_gradients_alone(H, N, block_q, rc, rm):
    """dK and dV of a slice, from a saved state, do not depend on how many others there are and when their workgroups start."""
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v, do = (torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(4))

    def grads(*xs):
        _, saved = sla.sla_attention_fwd_train(*xs[:3], block_q, 64, rc, rm)
        return sla.sla_attention_bwd(*xs, block_q, 64, rc, rm, saved=saved)[1:3]

    whole = grads(q, k, v, do)
    pick = [0, 3, H - 1]
    few = grads(*(x[:, pick].contiguous() for x in (q, k, v, do)))
    for a, b in zip(whole, few):
        assert torch.isfinite(b).all()
        assert torch.equal(a[:, pick], b)


@pytest.mark.parametrize("H, N, block_q, rc, rm", [
    (3, 129, 128, 0.34, 0.66),   # a query block of one row: the second workgroup of dQ has none
    (9, 4033, 128, 0.1, 0.2),    # dK/dV's workgroups in the order of their lists' lengths, dQ's behind them
    (7, 1000, 64, 0.2, 0.4),     # one workgroup of dQ per query block
    (15, 1000, 128, 0.2, 0.0),   # 240 half query blocks, no linear branch
    (4, 9000, 128, 0.4, 0.2),    # long lists, 568 workgroups of dQ: their second turn nearly empty, one launch
    (6, 9000, 128, 0.4, 0.2),    # 852: two launches
])
def test_gradients_of_one_launch_and_of_two_have_the_same_bits(H, N, block_q, rc, rm):
    """Calls of few query blocks form dQ in the launch of dK and dV, dq wherever its caller wants it."""
    many = 1024 // ((N + block_q - 1) // block_q * (block_q // 64)) + 1
    q, k, v, do = _qkv(many, N) + _qkv(many, N, seed=5)[:1]
    args = (block_q, 64, rc, rm)
    two = sla.sla_attention_bwd(q, k, v, do, *args, proj_w=_weight(0))[:3]
    few = [x[:, :H].contiguous() for x in (q, k, v, do)]
    one = sla.sla_attention_bwd(*few, *args, proj_w=_weight(0))[:3]
    token_major = torch.empty((1, N, H, D), dtype=torch.bfloat16, device="cuda").permute(0, 2, 1, 3)
    strided = (token_major, torch.empty_like(few[0]), torch.empty_like(few[0]))
    sla.sla_attention_bwd_strided(*few, *strided, *args, proj_w=_weight(0))
    for a, b, c in zip(two, one, strided):
        assert torch.isfinite(b).all()
        assert torch.equal(a[:, :H], b)
        assert torch.equal(c, b)
