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
    (25, 64, 1.0, 0.0, None),     # one short key block, no linear branch
    (81, 128, 0.5, 0.5, 0),       # two key blocks, the projection aligned
    (189, 64, 0.34, 0.66, 1),     # three query blocks (one wavefront of the four without a row), W off by two bytes
    (1000, 128, 0.2, 0.4, None),  # a ragged last key block, no projection
    (4033, 64, 0.1, 0.2, 1),      # 64 key blocks, the last of one token: the longest slice of the one-launch route
    (4097, 128, 0.1, 0.2, 0),     # 65: the shortest of the other
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
