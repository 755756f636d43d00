"""The epilogue and its reverse mode, and the gates' reverse mode, against plain
torch in fp64: row widths at the edges of the quads-per-lane steps (1 to 16) and
of the column sum's 32-column groups, row counts around its 32 parts, and heads
whose tokens are fewer and more than one workgroup's threads, of one sequence
and of many."""
import pytest
import torch

from paper_2607_07386_amd import sdm
from tests.gpu_util import DEV, REGRESSION_TOL

pytestmark = pytest.mark.gpu


def rel(a, b):
    return ((a.double() - b).abs().max() / b.abs().max().clamp_min(1e-30)).item()


@pytest.mark.parametrize("act", [0, 1])
@pytest.mark.parametrize("T,d_v", [(1, 4), (37, 36), (2100, 128), (300, 256), (70, 260), (40, 516), (40, 1028),
                                   (33, 2048), (9, 2052), (5, 4096)])
def test_epilogue_widths(T, d_v, act):
    g = torch.Generator(device=DEV).manual_seed(T + d_v)
    n = lambda *s: torch.randn(s, generator=g, device=DEV)
    y, gate, gamma, dout = n(2, 3, T, d_v), n(2, 3, T, d_v).bfloat16(), n(d_v), n(2, 3, T, d_v)
    o, rstd = sdm.norm_gate(y, gate, gamma, 1e-5, act, want_rstd=True)
    dy, dg, dgamma = sdm.norm_gate_bwd(y, gate, gamma, 1e-5, act, dout)
    yd, gd, md = (t.double().requires_grad_() for t in (y, gate, gamma))
    r = torch.rsqrt(yd.square().mean(-1, keepdim=True) + 1e-5)
    ref = yd * r * md * (torch.nn.functional.silu(gd) if act else gd)
    gy, gg, gm = torch.autograd.grad(ref, (yd, gd, md), dout.double())
    for a, b in ((o, ref), (rstd, r[..., 0]), (dy, gy), (dg, gg), (dgamma, gm)):
        assert rel(a, b.detach()) <= REGRESSION_TOL


@pytest.mark.parametrize("B,H,T", [(1, 1, 1), (3, 2, 7), (2, 3, 1025), (1, 5, 2500), (1500, 3, 1),
                                   (70, 2, 37), (5, 2, 1024), (3, 2, 2048)])
def test_gates_bwd_sums(B, H, T):
    g = torch.Generator(device=DEV).manual_seed(T)
    n = lambda *s: torch.randn(s, generator=g, device=DEV)
    a, b, da, db = n(B, H, T), n(B, H, T), n(B, H, T), n(B, H, T)
    A, bdt = n(H).abs(), n(H)
    got = sdm.gates_bwd(a, b, A, bdt, da, db)
    ad, bd, Ad, td = (t.double().requires_grad_() for t in (a, b, A, bdt))
    al = torch.exp(-Ad[:, None] * torch.nn.functional.softplus(ad + td[:, None]))
    ref = torch.autograd.grad((al, bd.sigmoid()), (ad, bd, Ad, td), (da.double(), db.double()))
    for x, r in zip(got, ref):
        assert rel(x, r) <= REGRESSION_TOL


@pytest.mark.parametrize("B,T", [(512, 32), (4096, 1), (64, 37)])
def test_gates_bwd_short_sequences_fill_the_workgroup(B, T):
    """The time depends on a head's tokens, not on how many sequences they come from:
    many short ones take about as long as one sequence of as many tokens (measured
    1.0 to 1.9 times, 5 to 200 where each sequence is a pass of its own)."""
    H = 8

    def micros(B, T):
        n = lambda *s: torch.randn(s, device=DEV)
        a, b, da, db, A, bdt = n(B, H, T), n(B, H, T), n(B, H, T), n(B, H, T), n(H).abs(), n(H)
        times = []
        for _ in range(9):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(4):
                sdm.gates_bwd(a, b, A, bdt, da, db)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1) * 250)
        return sorted(times)[4]

    # launches back to back take about 15 us whatever they do
    assert micros(B, T) <= 3 * max(micros(1, B * T), 15)


def test_gates_bwd_without_tokens():
    z = torch.zeros((2, 3, 0), device=DEV)
    dA, db_dt = sdm.gates_bwd(z, z, torch.ones(3, device=DEV), torch.ones(3, device=DEV), z, z)[2:]
    assert not dA.any() and not db_dt.any()
