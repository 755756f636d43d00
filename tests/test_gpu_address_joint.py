"""Both sides' addressing in one launch (a first stage that runs alone) against
sdm_address on each side, bit for bit: list lengths that differ, each addressing
mode and kernel (tiles, half by half, scores in registers), and pairs of lengths
that need different kernels and so keep two launches."""
import pytest
import torch

from paper_2607_07386_amd import sdm
from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu


# (sqrt(N), d_k, W, R, dtype, direct)
CASES = [(20, 16, 4, 7, torch.float32, False), (130, 48, 32, 9, torch.bfloat16, False),
         (300, 64, 8, 20, torch.bfloat16, False), (600, 128, 32, 32, torch.bfloat16, False),
         (640, 72, 40, 64, torch.bfloat16, False), (48, 96, 48, 33, torch.bfloat16, True),
         (48, 96, 48, 24, torch.float32, True), (140, 32, 100, 70, torch.bfloat16, False),
         (140, 32, 100, 32, torch.bfloat16, False)]


@pytest.mark.parametrize("s,d_k,W,R,dtype,direct", CASES)
def test_joint_addressing(s, d_k, W, R, dtype, direct):
    B, H, T, d_v = 1, 3, 39, 8
    g = torch.Generator(device=DEV).manual_seed(s + W)
    n = lambda *sh: torch.randn(sh, generator=g, device=DEV)
    q, k, v, gate = n(B, H, T, d_k).to(dtype), n(B, H, T, d_k).to(dtype), n(B, H, T, d_v).to(dtype), n(B, H, T, d_v).to(dtype)
    a, b = n(B, H, T).to(dtype), n(B, H, T).to(dtype)
    cbq, cbk = (None, None) if direct else (n(H, 2, s, d_k // 2).to(dtype), n(H, 2, s, d_k // 2).to(dtype))
    mem = torch.zeros((B, H, s * s, d_v), device=DEV)
    ws = sdm.fwd_workspace(B, H, T, W, R, DEV)
    ws[:16] = 255   # stale error words: cleared by the call
    o = sdm.layer_fwd(q, k, cbq, cbk, v, a, b, gate, n(H).abs(), n(H), None, 1e-5, 1, mem, s * s, W, R, workspace=ws)
    sdm.check_device_errors(ws)
    ri, rv = sdm.address(q, cbq, s * s, R)
    wi, wv = sdm.address(k, cbk, s * s, W)
    for got, ref in ((o["r_idx"], ri), (o["r_val"], rv), (o["w_idx"], wi), (o["w_val"], wv)):
        assert torch.equal(got, ref)
