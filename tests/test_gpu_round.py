"""The forward scan in rounds of tokens against the oracle: list lengths at the
edges of its rows-per-lane steps, row widths that leave lanes of the last column
group without columns, sequences that end inside a round, lists from so few slots that most tokens
share some (waits inside a round, ring rows of earlier rounds) and from so many
that few do, with and without the undo log; with helper workgroups, which must
not change a bit; and which shapes take it."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_07386_amd import sdm
from tests.gpu_util import DEV, REGRESSION_TOL, rel_err

pytestmark = pytest.mark.gpu

# (streams, T, N, W, R, d_v, slots in use): tables of N slots that the dispatch gives to
# this kernel, and lists drawn from fewer of them (evenly spread), so that tokens chain
SHAPES = {
    "one-row": (3, 37, 5, 1, 1, 32, 5),
    "k1-full": (2, 200, 40, 8, 8, 64, 40),
    "k1-odd": (3, 41, 30, 7, 3, 36, 30),
    "k2": (2, 65, 64, 16, 16, 32, 64),
    "k2-odd": (2, 50, 64, 9, 15, 100, 64),
    "k4-dense": (2, 150, 3072, 32, 32, 64, 40),
    "k4-sparse": (16, 160, 4096, 32, 32, 32, 4096),
    "k4-mixed": (3, 77, 2401, 32, 17, 128, 200),
    "k8-dense": (2, 130, 16384, 64, 64, 32, 80),
    "k8-sparse": (8, 131, 16384, 64, 64, 64, 9000),
    "k8-mixed": (3, 53, 10368, 48, 24, 100, 300),
    "k8-edge": (2, 4, 18818, 33, 64, 44, 99),
}


def _lists(rng, S, T, N, k, use):
    ids = np.sort(rng.choice(N, use, replace=False))
    return np.stack([np.stack([ids[np.sort(rng.choice(use, k, replace=False))] for _ in range(T)])
                     for _ in range(S)]).astype(np.int32)


def _other_kernel(fn):
    """fn() by the kernels of a forced geometry, which never go in rounds."""
    sdm.set_scan_prefetch(4)
    try:
        return fn()
    finally:
        sdm.set_scan_prefetch(0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("name", list(SHAPES))
def test_round_scan(name, dtype):
    S, T, N, W, R, dv, use = SHAPES[name]
    rng = np.random.default_rng(1000 + len(name) * 7 + W + R)
    wi, ri = _lists(rng, S, T, N, W, use), _lists(rng, S, T, N, R, use)
    wv = (rng.random((S, T, W)) * 2 / np.sqrt(W)).astype(np.float32)
    rv = rng.random((S, T, R)).astype(np.float32)
    dev = lambda a, dt=None: torch.from_numpy(np.ascontiguousarray(a))[:, None].to(DEV, dt)
    v, al, be = (dev(x.astype(np.float32), dtype) for x in (rng.standard_normal((S, T, dv)), rng.uniform(0.1, 1, (S, T)),
                                                            rng.uniform(0.1, 1, (S, T))))
    m0 = rng.standard_normal((S, N, dv)).astype(np.float32)
    f64 = lambda t: t[:, 0].double().cpu().numpy()
    memo = m0.astype(np.float64)
    yo, so = oracle.scan_fwd(wi, wv, ri, rv, f64(v), f64(al), f64(be), memo, save=True)

    def run(save):
        mem, saved = dev(m0), sdm.saved_buffer(S, 1, T, W, dv, DEV) if save else None
        y = sdm.scan_fwd(dev(wi), dev(wv), dev(ri), dev(rv), v, al, be, mem, saved=saved)
        torch.cuda.synchronize()
        return y, mem, saved

    y, mem, saved = run(True)
    # fp32 sums of up to 64 terms on both sides of the recurrence
    for got, ref in ((y, yo), (mem, memo), (saved, so)):
        assert rel_err(f64(got), np.asarray(ref).reshape(f64(got).shape)) <= REGRESSION_TOL
    y2, mem2, _ = run(False)
    assert torch.equal(y, y2) and torch.equal(mem, mem2)
    # the sums over rows are in another order there: the same bits would mean the same kernel
    if W > 1:
        assert not torch.equal(y, _other_kernel(lambda: run(False))[0])


def test_round_scan_stages_and_helpers():
    """Stages of 64 tokens (no helpers) and one stage of 700 (helpers) of the same
    call: the same bits, also against a table row's value carried over a stage."""
    B, H, T, s, k, d = 1, 4, 700, 64, 32, 64
    g = torch.Generator(device=DEV).manual_seed(5)
    n = lambda *sh: torch.randn(sh, generator=g, device=DEV)
    q, kk, v = (n(B, H, T, d).bfloat16() for _ in range(3))
    al, be = (torch.sigmoid(n(B, H, T)).bfloat16() for _ in range(2))
    cb = n(H, 2, s, d // 2).bfloat16()
    out = []
    for chunk in (0, 64, 192):
        mem = torch.zeros((B, H, s * s, d), device=DEV)
        o = sdm.forward(q, kk, cb, cb, v, al, be, mem, s * s, k, chunk=chunk)
        torch.cuda.synchronize()
        out.append((o["y"], mem))
    for y, mem in out[1:]:
        assert torch.equal(y, out[0][0]) and torch.equal(mem, out[0][1])


def test_round_scan_two_gib_of_output():
    """A stream whose y ends just below 2 GiB, at a length that leaves waves of the last
    rounds without a token: those tokens' offsets lie past 2 GiB, and what is stored
    for them must not land in y's first rows."""
    T, N, k, dv, head = 559239, 64, 8, 960, 64
    assert T * dv * 4 < 2 ** 31 <= (T + 8) * dv * 4
    g = torch.Generator(device=DEV).manual_seed(3)
    lists = lambda: (torch.randint(0, N // k, (1, 1, T, k), generator=g, device=DEV) +
                     torch.arange(k, device=DEV) * (N // k)).int()
    u = lambda *sh: torch.rand(sh, generator=g, device=DEV)
    args = [lists(), u(1, 1, T, k) / k, lists(), u(1, 1, T, k),
            torch.randn((1, 1, T, dv), generator=g, device=DEV, dtype=torch.bfloat16), u(1, 1, T).bfloat16(),
            u(1, 1, T).bfloat16()]
    y = sdm.scan_fwd(*args, torch.zeros((1, 1, N, dv), device=DEV))[:, :, :head].clone()
    short = sdm.scan_fwd(*(a[:, :, :head].contiguous() for a in args), torch.zeros((1, 1, N, dv), device=DEV))
    torch.cuda.synchronize()
    assert torch.equal(y, short)


@pytest.mark.parametrize("T", [130, 2100])
def test_chunked_call_in_rounds(T):
    """sdm_scan_fwd_chunked on a table large enough for the scan in rounds (one range,
    and eight ranges with a ragged end): the oracle's recurrence, with forget gates of
    zero and below taken as 1e-30 and flagged, as the chunk form does."""
    S, N, W, dv = 2, 20480, 32, 32
    rng = np.random.default_rng(T)
    wi = np.sort(rng.integers(0, N // W, (S, T, W)) + np.arange(W) * (N // W), -1).astype(np.int32)
    ri = np.where(rng.random((S, T, W)) < 0.3, wi, np.roll(wi, 1, axis=1)).astype(np.int32)
    wv, rv = (rng.random((S, T, W)) / 8).astype(np.float32), rng.random((S, T, W)).astype(np.float32)
    v, be = rng.standard_normal((S, T, dv)).astype(np.float32), rng.random((S, T)).astype(np.float32)
    al = rng.uniform(0.1, 1, (S, T)).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a))[:, None].to(DEV)
    ws = sdm.chunked_workspace(S, 1, T, W, W, DEV)
    for bad in (False, True):
        if bad:
            al[0, 40], al[1, 77] = 0.0, -0.5
        mem, memo = torch.zeros((S, 1, N, dv), device=DEV), np.zeros((S, N, dv))
        sdm.profile_enable(True)
        y = sdm.scan_fwd_chunked(dev(wi), dev(wv), dev(ri), dev(rv), dev(v), dev(al), dev(be), mem, workspace=ws)
        torch.cuda.synchronize()
        assert sdm.profile_read("chunk_scan")[1] == 0 and sdm.profile_read("fwd_scan")[1] == (8 if T > 2047 else 1)
        sdm.profile_enable(False)
        yo = oracle.scan_fwd(wi, wv, ri, rv, v, np.maximum(al, 1e-30), be, memo)
        assert rel_err(y[:, 0].cpu().numpy(), yo) <= REGRESSION_TOL
        assert rel_err(mem[:, 0].cpu().numpy(), memo) <= REGRESSION_TOL
        if bad:
            with pytest.raises(sdm.SdmError) as e:
                sdm.check_device_errors(ws)
            assert e.value.status == -5 and "alpha" in str(e.value)
        else:
            sdm.check_device_errors(ws)


@pytest.mark.parametrize("S,N,W,R,dv,rounds", [
    (16, 1279, 8, 8, 128, 0), (16, 1280, 8, 8, 128, 1), (16, 20479, 32, 32, 128, 0), (16, 20480, 32, 32, 128, 1),
    (8, 3200, 8, 32, 128, 0), (8, 20480, 8, 32, 128, 1), (32, 3200, 8, 32, 128, 1),     # narrow or wide chunk kernel
    (65, 20480, 32, 32, 128, 0),                                                        # the line kernel's from here on
    (8, 65535, 40, 40, 128, 0), (8, 65536, 40, 40, 128, 1), (32, 16383, 48, 24, 128, 0), (32, 16384, 48, 24, 128, 1),
    (16, 16383, 56, 56, 128, 0), (16, 16384, 56, 56, 128, 1), (512, 4095, 40, 40, 32, 0), (512, 4096, 40, 40, 32, 1),
    (32, 131071, 8, 64, 32, 0), (32, 131072, 8, 64, 32, 1), (32, 32767, 32, 64, 32, 0),
    (32, 32768, 32, 64, 32, 1), (4, 8191, 64, 64, 128, 0), (4, 8192, 64, 64, 128, 1)])
def test_which_chunked_calls_go_in_rounds(S, N, W, R, dv, rounds):
    """The chunk form keeps the tables on which tokens of a round share slots."""
    T = 64
    g = torch.Generator(device=DEV).manual_seed(N)
    u = lambda *sh: torch.rand(sh, generator=g, device=DEV)
    lists = lambda k: (torch.randint(0, N // k, (1, S, T, k), generator=g, device=DEV) +
                       torch.arange(k, device=DEV) * (N // k)).int()
    args = (lists(W), u(1, S, T, W) / W, lists(R), u(1, S, T, R), u(1, S, T, dv), u(1, S, T) / 2 + 0.5, u(1, S, T))
    mem = torch.zeros((1, S, N, dv), device=DEV)
    sdm.profile_enable(True)
    y = sdm.scan_fwd_chunked(*args, mem)
    torch.cuda.synchronize()
    ran = sdm.profile_read("fwd_scan")[1], sdm.profile_read("chunk_scan")[1]
    sdm.profile_enable(False)
    assert ran == ((1, 0) if rounds else (0, 1))
    mem2 = torch.zeros_like(mem)
    y2 = sdm.scan_fwd(*args, mem2)
    for a, b in ((y, y2), (mem, mem2)):
        assert ((a - b).abs().max() / b.abs().max()).item() <= REGRESSION_TOL


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("name", list(SHAPES))
def test_round_backward(name, dtype):
    """The backward in rounds on the same shapes: every gradient against the oracle's
    reverse pass, the table restored bit for bit, and stages of 64 tokens giving the
    same bits as one stage."""
    S, T, N, W, R, dv, use = SHAPES[name]
    rng = np.random.default_rng(2000 + len(name) * 7 + W + R)
    wi, ri = _lists(rng, S, T, N, W, use), _lists(rng, S, T, N, R, use)
    wv = (rng.random((S, T, W)) * 2 / np.sqrt(W)).astype(np.float32)
    rv = rng.random((S, T, R)).astype(np.float32)
    dev = lambda a, dt=None: torch.from_numpy(np.ascontiguousarray(a))[:, None].to(DEV, dt)
    v, al, be = (dev(x.astype(np.float32), dtype) for x in (rng.standard_normal((S, T, dv)), rng.uniform(0.1, 1, (S, T)),
                                                            rng.uniform(0.1, 1, (S, T))))
    m0, dy = rng.standard_normal((S, N, dv)).astype(np.float32), rng.standard_normal((S, T, dv)).astype(np.float32)
    dmT = rng.standard_normal((S, N, dv)).astype(np.float32)
    f64 = lambda t: t[:, 0].double().cpu().numpy()
    memo = m0.astype(np.float64)
    _, so = oracle.scan_fwd(wi, wv, ri, rv, f64(v), f64(al), f64(be), memo, save=True)
    go = oracle.scan_bwd(wi, wv, ri, rv, f64(v), f64(al), f64(be), memo, so, dy.astype(np.float64),
                         dmem_T=dmT.astype(np.float64))
    args = (dev(wi), dev(wv), dev(ri), dev(rv), v, al, be)
    mem, saved = dev(m0), sdm.saved_buffer(S, 1, T, W, dv, DEV)
    sdm.scan_fwd(*args, mem, saved=saved)
    mem_T = mem.clone()
    got = []
    for chunk in (T, 64):
        mem.copy_(mem_T)
        got.append(sdm.scan_bwd(*args, mem, saved, dev(dy), dmem_T=dev(dmT), want_dqk=False, chunk=chunk))
        torch.cuda.synchronize()
        assert torch.equal(mem, dev(m0))
    mem.copy_(mem_T)
    other = _other_kernel(lambda: sdm.scan_bwd(*args, mem, saved, dev(dy), dmem_T=dev(dmT), want_dqk=False))
    assert not all(torch.equal(got[0][k], other[k]) for k in other if other[k] is not None)
    for k in ("dv", "dalpha", "dbeta", "dmem0", "dw_val", "dr_val"):
        assert torch.equal(got[0][k], got[1][k]), k
        assert rel_err(f64(got[0][k]), np.asarray(go[k]).reshape(f64(got[0][k]).shape)) <= REGRESSION_TOL, k


@pytest.mark.parametrize("S,N,k,plain,log,bwd,dv", [(130, 4607, 48, 0, 1, 0, 36), (130, 4608, 48, 1, 1, 0, 36), (130, 6144, 48, 1, 1, 1, 36),
                                                     (512, 6144, 48, 1, 1, 0, 36)] + [t + (32,) for t in [
    # workgroups: 4 below one per compute unit, 260 above one, 520 above two
    (4, 16, 8, 1, 1, 1), (520, 16, 8, 1, 1, 1),                                  # up to 8 rows: any table
    (4, 32, 16, 1, 1, 1), (260, 32, 16, 1, 1, 0), (520, 136, 16, 0, 0, 0),       # up to 16: but dense ones by many streams
    (520, 341, 16, 0, 1, 0), (520, 342, 16, 1, 1, 0), (520, 1024, 16, 1, 1, 1),
    (4, 863, 24, 0, 0, 0), (4, 864, 24, 1, 1, 0), (4, 2304, 24, 1, 1, 1),
    (260, 921, 24, 0, 0, 0), (260, 2303, 24, 0, 1, 0), (260, 2304, 24, 1, 1, 1),
    (4, 7679, 48, 0, 0, 0), (4, 7680, 48, 1, 1, 0), (4, 15359, 48, 1, 1, 0), (4, 15360, 48, 1, 1, 1),
    (260, 9215, 48, 0, 1, 0), (260, 9216, 48, 1, 1, 0), (260, 12288, 48, 1, 1, 1),
    (4, 3071, 32, 0, 0, 0), (4, 3072, 32, 1, 1, 1),                              # the line kernel's lists
    (4, 12287, 64, 0, 0, 0), (4, 12288, 64, 1, 1, 0), (4, 16384, 64, 1, 1, 1)]])
def test_which_scans_go_in_rounds(S, N, k, plain, log, bwd, dv):
    """Tables on which the tokens of a round wait for each other keep the other scan
    kernels, without and with the undo log and in the backward: their bits are a forced
    geometry's there, and only there (the sums over rows are in another order).  A
    workgroup per stream with d_v = 32, two with 36."""
    T = 32
    g = torch.Generator(device=DEV).manual_seed(S + N + k)
    u = lambda *sh: torch.rand(sh, generator=g, device=DEV)
    lists = lambda: (torch.randint(0, N // k, (1, S, T, k), generator=g, device=DEV) +
                     torch.arange(k, device=DEV) * (N // k)).int()
    args = (lists(), u(1, S, T, k) / k, lists(), u(1, S, T, k), u(1, S, T, dv) - 0.5, u(1, S, T), u(1, S, T))
    dy = u(1, S, T, dv) - 0.5

    def scans():
        y = sdm.scan_fwd(*args, torch.zeros((1, S, N, dv), device=DEV))
        mem, saved = torch.zeros((1, S, N, dv), device=DEV), sdm.saved_buffer(1, S, T, k, dv, DEV)
        y_log = sdm.scan_fwd(*args, mem, saved=saved)
        # the backward from one state, whichever kernel ran before
        mem.zero_()
        sdm.set_scan_line_io(False)
        try:
            sdm.scan_fwd(*args, mem, saved=saved)
        finally:
            sdm.set_scan_line_io(True)
        gr = sdm.scan_bwd(*args, mem, saved, dy, want_dqk=False)
        return y, y_log, torch.cat([gr[n].flatten() for n in ("dv", "dalpha", "dw_val", "dr_val")])

    same = [torch.equal(a, b) for a, b in zip(scans(), _other_kernel(scans))]
    assert same == [not plain, not log, not bwd]
