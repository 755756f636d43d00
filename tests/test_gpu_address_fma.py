"""Codebook scoring without matrix cores (fp32, and bf16 halves that are not
multiples of eight): token counts around the eight-token groups of a thread and
the tile heights, odd depths, and list lengths on either side of 32 and 64,
against a choice from 64-bit scores rounded to fp32."""
import pytest
import torch

from paper_2607_07386_amd import sdm
from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,s,dh,k", [(1, 9, 1, 3), (7, 64, 5, 33), (9, 65, 12, 64), (17, 130, 37, 16), (25, 300, 3, 20),
                                      (8, 600, 18, 70), (33, 33, 23, 33), (16, 128, 100, 128)])
def test_fma_scores(T, s, dh, k, dtype):
    g = torch.Generator(device=DEV).manual_seed(s + dh)
    x = torch.randn((2, 2, T, 2 * dh), generator=g, device=DEV).to(dtype)
    cb = torch.randn((2, 2, s, dh), generator=g, device=DEV).to(dtype)
    idx, val, score = sdm.address(x, cb, s * s, k, want_score=True)
    sub = [torch.einsum("bhtd,hjd->bhtj", x[..., h * dh:(h + 1) * dh].double(), cb[:, h].double()) for h in (0, 1)]
    full = (sub[0].float()[..., :, None] + sub[1].float()[..., None, :]).flatten(-2).double()
    # every selected slot carries its own score, and no slot left out beats the last one taken (to fp32 sums'
    # rounding: dh terms of size about one)
    tol = 2e-6 * dh ** 0.5 * 4
    assert (full.gather(-1, idx.long()) - score.double()).abs().max() <= tol
    assert (idx[..., 1:] > idx[..., :-1]).all()
    kth = full.topk(k, dim=-1).values[..., -1]
    assert (score.double().min(-1).values - kth).abs().max() <= tol
    assert (val.double() - torch.softmax(score.double(), -1)).abs().max() <= 1e-6


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("s,dh,k", [(9, 1, 3), (64, 5, 33), (130, 18, 16), (300, 37, 20), (600, 100, 70), (1024, 3, 128)])
def test_one_token_scores_as_many(s, dh, k, dtype):
    """The decode step scores its single token by threads of one token, the tiles by
    threads of eight: the same chains, so the same bits, also as in a tile of nine."""
    g = torch.Generator(device=DEV).manual_seed(s + dh)
    B, H, d_v = 2, 2, 8
    x = torch.randn((B, H, 9, 2 * dh), generator=g, device=DEV).to(dtype)
    cb = torch.randn((H, 2, s, dh), generator=g, device=DEV).to(dtype)
    many = sdm.address(x, cb, s * s, k, want_score=True)
    one = x[:, :, :1].contiguous()
    for a, b in zip(sdm.address(one, cb, s * s, k, want_score=True), many):
        assert torch.equal(a, b[:, :, :1])
    z = torch.ones((B, H, 1), device=DEV).to(dtype)
    o = sdm.forward(one, one, cb, cb, torch.zeros((B, H, 1, d_v), device=DEV).to(dtype), z, z,
                    torch.zeros((B, H, s * s, d_v), device=DEV), s * s, k)
    for name, b in (("r_idx", many[0]), ("r_val", many[1]), ("w_idx", many[0]), ("w_val", many[1])):
        assert torch.equal(o[name], b[:, :, :1])
