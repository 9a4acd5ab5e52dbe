"""GPU parity of the forward on its long tiles, at sizes where these can go wrong, against the fp64 oracle through the C ABI:
256 tokens x 32 lanes in fp32, 128 x 64 with the harmonic convolution (bf16 without it: test_gpu_bf16).  4200 tokens are
more than the 64-token tiles are taken for.  Up to 768 - 2048 tiles a call has a workgroup for every tile, whose threads read
their rows themselves; beyond that workgroups take several, staged ahead in LDS, and in fp32 on 32-lane rows pass a prefix on
per tile instead of per group of tiles.  Bar as in the other parity tests; gate masks bit for bit."""
import numpy as np
import pytest

from oracle import cawn_oracle as O

pytestmark = pytest.mark.gpu

TOL = 1e-4
L = 4200


def _gpu():
    import gpu_util
    return gpu_util


def _check(B, H, F, Kc, valve=False, ret=False, hconv=False, bf16=False, concat=False, seed=0, L=L, ws=None):
    """A call that continues a sequence: outputs, gate mask, carried state and checkpoints."""
    G = _gpu()
    r = np.random.Generator(np.random.PCG64(9000 + seed + 131 * H + F + Kc))
    J, kk = H * F, max(Kc, 1)
    n = lambda *s: r.standard_normal(s, dtype=np.float32)
    ex = G.bf16_exact if bf16 else (lambda x: x)
    d = dict(mag=ex(n(B, L, J)), ang=ex(n(B, L, J)), gamma=r.uniform(0.9, 0.9999, J).astype(np.float32),
             theta=r.uniform(0, np.pi, J).astype(np.float32), conv_w=n(2, J, kk) / np.float32(np.sqrt(kk)),
             conv_b=0.1 * n(2, J))
    scan, tail = n(B, 2, J), n(B, max(Kc - 1, 0), 2, J)
    mode = dict(valve=-3.9 + 3.0 * n(B, L, H) if valve else None,
                ret=1.0 + 1.5 * n(B, L, H) if ret else None, ret_bias=np.linspace(3.0, 0.0, F, dtype=np.float32) if ret else None)
    hc = dict(hconv_w=n(2, H, 3), hconv_b=n(2, H)) if hconv else {}
    tau, amp = (0.0, 1) if valve else (0.25, 0)
    ora = O.phase_fwd(O.Cfg(B, L, H, F, conv_k=Kc, amp_mode=amp, gate_mode=int(valve), gate_tau=tau, ret_mode=int(ret)),
                      d["mag"], d["ang"], None if ret else d["gamma"], d["theta"], conv_w=d["conv_w"], conv_b=d["conv_b"],
                      scan_in=scan.astype(np.float64), tail_in=tail if Kc > 1 else None, **mode)
    out = G.run_fwd(d, B, L, H, F, conv_k=Kc, amp_mode=amp, gate_tau=tau, want_ckpt=True, concat=concat, bf16=bf16, ws=ws,
                    state_in=G.pack_state(scan, tail if Kc > 1 else None), **mode, **hc)
    z = (ora["z_re"], ora["z_im"])
    # (a checkpoint is the unclamped state before every eighth token, the oracle's output that state unless it was clamped)
    planes = np.stack(z, 2)
    before = np.concatenate([scan[:, None].astype(np.float64), planes[:, 7:L - 1:8]], 1)
    free = np.abs(before) < 100.0
    assert free.mean() > 0.99
    if hconv:
        z = O.harmonic_conv(z[0], z[1], H, F, hc["hconv_w"], hc["hconv_b"])
    for k, want in (("z_re", z[0]), ("z_im", z[1])):
        e = G.bf16_err(out[k], want) if bf16 else G.rel_err(out[k], want) / TOL
        assert e <= 1.0, (k, e)
    assert np.array_equal(out["mask"], G.mask_from_gate(ora["gate"])), "gate mask differs"
    assert G.rel_err(out["ckpt"].reshape(before.shape)[free], before[free]) <= TOL
    s, t = G.unpack_state(out["state_out"], B, J, Kc)
    assert G.rel_err(s, ora["scan_out"]) <= TOL
    if Kc > 1:
        assert np.array_equal(t, ora["tail_out"])


# lanes that are no multiple of 4 or of 32 (a ragged last block, a last mask word); few tiles, more than the chip holds
# workgroups at a time (561 and 544), and workgroups that take several (1071 and 1037: staged word by word)
@pytest.mark.parametrize("B,H,F", [(1, 1, 65), (2, 5, 24), (11, 1, 66), (32, 1, 30), (21, 1, 66), (61, 1, 30)])
@pytest.mark.parametrize("Kc", [0, 2, 4])
def test_long_tiles_odd_lanes(B, H, F, Kc):
    _check(B, H, F, Kc, concat=Kc == 2)


# heads of a quarter, half, all and three of a 32-lane row; then 33 chains of 17 tiles, a workgroup each but with
# retentions; the last three: workgroups that take several (1054, 1037 and 1071 tiles), with a last block that is half, three quarters and wholly full
@pytest.mark.parametrize("valve,ret", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("B,H,F", [(1, 5, 8), (1, 3, 16), (2, 1, 96), (11, 3, 32), (31, 3, 16), (61, 3, 8), (21, 3, 32)])
def test_long_tiles_valve_and_retention(B, H, F, valve, ret):
    if valve and ret and F < 16:
        pytest.skip("heads of 8 with both logits are refused")
    _check(B, H, F, 3, valve=valve, ret=ret, seed=1)


# heads inside a 64-lane row, of exactly one, of two and of four; then 528 tiles, more than the chip holds workgroups at a time,
# and heads of two blocks, more than workgroups that take them; the last two: workgroups that take several tiles (1848, 1815),
# with a last row that is full and one that is three quarters full
@pytest.mark.parametrize("B,H,F", [(1, 5, 4), (1, 3, 16), (1, 3, 32), (2, 3, 64), (1, 3, 128), (1, 3, 256), (8, 2, 64), (8, 2, 128),
                                   (28, 2, 64), (55, 3, 16)])
@pytest.mark.parametrize("bf16", [False, True])
def test_long_tiles_harmonic_convolution(B, H, F, bf16):
    _check(B, H, F, 3, hconv=True, bf16=bf16, concat=F == 16, seed=2)


# ... and the last: workgroups that take several of 2112 tiles, a second row of lanes that is half full
@pytest.mark.parametrize("valve,ret", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("B,H,F", [(1, 3, 32), (1, 2, 64), (1, 2, 128), (1, 1, 256), (8, 2, 64), (32, 3, 32)])
@pytest.mark.parametrize("bf16", [False, True])
def test_long_tiles_harmonic_convolution_with_logits(B, H, F, valve, ret, bf16):
    _check(B, H, F, 3, valve=valve, ret=ret, hconv=True, bf16=bf16, seed=3)


# Either side of the lines between a workgroup for every tile and workgroups that take several (17 and 33 tiles a chain, 256
# compute units): 32-lane rows 768 tiles, 1024 where the chains are a multiple of four or a head has logits; 64-lane rows 1792,
# 2048 with retentions (bf16 without the harmonic convolution: test_gpu_bf16).  The first of each pair has more tiles than the
# chip holds workgroups of its kernel at a time.
@pytest.mark.parametrize("B,F,valve,ret,hconv,bf16", [
    (45, 24, False, False, False, False), (46, 24, False, False, False, False), (60, 24, False, False, False, False), (61, 24, False, False, False, False),
    (45, 32, True, False, False, False), (47, 32, True, False, False, False),
    (60, 32, True, False, False, False), (61, 32, True, False, False, False), (60, 32, False, True, False, False), (61, 32, False, True, False, False),
    (60, 32, True, True, False, False), (61, 32, True, True, False, False),
    (54, 64, False, False, True, False), (55, 64, False, False, True, False), (62, 64, True, True, True, False), (63, 64, True, True, True, False),
    (54, 64, True, False, True, True), (55, 64, True, False, True, True),
    (62, 32, True, True, True, True), (63, 32, True, True, True, True)])
def test_long_tiles_around_the_line_between_one_and_several_a_workgroup(B, F, valve, ret, hconv, bf16):
    _check(B, 1, F, 3, valve=valve, ret=ret, hconv=hconv, bf16=bf16, seed=4)


# ... and 64-lane rows with both logits: 3072 tiles in fp32 and 4096 in bf16 (33 tiles a chain)
@pytest.mark.parametrize("B,hconv,bf16", [(93, True, False), (94, True, False), (124, True, True), (125, True, True), (124, False, True), (125, False, True)])
def test_long_tiles_around_the_line_with_both_logits(B, hconv, bf16):
    if hconv:
        _check(B, 1, 64, 1, valve=True, ret=True, hconv=True, bf16=bf16, seed=6)
    else:
        import test_gpu_bf16 as T
        T._check_fwd(B, L, 1, 64, 2, T._inputs(B, L, 1, 64, 2, 9600), amp_mode=1, valve=True, ret=True)


# ... with few chains: 5 and 7 of 159 and 113 tiles (a workgroup for each of 795, several of 791 a workgroup), 14 and 18 of 57 and 44
# (798, 792); an odd number of chains with a few tiles more than the chip holds workgroups (33 of 17; 17 of 32; 25 of 33 where
# 768 fit) and a few more still (35; 19); rows of 64 lanes without a conv, chains of 33
# tiles around 1280 (38, 39) and, with retentions, 1792 (54, 55)
@pytest.mark.parametrize("B,L,F,Kc,valve,ret,hconv", [
    (5, 40600, 24, 3, False, False, False), (7, 28800, 24, 3, False, False, False), (14, 14500, 32, 3, True, False, False),
    (18, 11200, 32, 3, True, False, False), (33, 4200, 32, 3, True, True, False), (35, 4200, 32, 3, True, True, False),
    (17, 4090, 64, 3, True, False, True), (19, 4090, 64, 3, True, False, True), (25, 4200, 64, 0, True, False, True),
    (38, 4200, 64, 0, False, False, True), (39, 4200, 64, 0, False, False, True), (54, 4200, 64, 0, False, True, True), (55, 4200, 64, 0, False, True, True)])
def test_long_tiles_few_chains_or_few_more_than_fit(B, L, F, Kc, valve, ret, hconv):
    _check(B, 1, F, Kc, valve=valve, ret=ret, hconv=hconv, seed=5, L=L)


# 64-token tiles, long tiles with a workgroup each, rows of 64 lanes; every one with more than 96 workgroups, which are counted
# out in two levels and draw from several counters
@pytest.mark.parametrize("B,L,H,F,hconv", [(4, 512, 12, 64, False), (1, 4200, 6, 64, False), (1, 4200, 4, 64, True)])
def test_a_call_that_gave_up_leaves_the_workspace_ready(B, L, H, F, hconv):
    """With a spin limit of zero, set from the host, every wait that is not already over gives up: the call drains, and the
    next one on the same workspace is right (tickets, counts and epoch were reset)."""
    G = _gpu()
    from paper_2604_04250_amd import binding as K
    import torch
    J = H * F
    d = K.make_desc(B, L, H, F, gate_tau=0.25, hconv_k=3 if hconv else 0)
    ws = torch.empty((K.cawn_workspace_bytes(K.make_desc(B, L, H, F, conv_k=3, hconv_k=d.hconv_k)) + 3) // 4,
                     dtype=torch.int32, device=G.DEV)
    K.check(K.cawn_workspace_init(ws))
    x, z = torch.randn((2, B, L, J), device=G.DEV), torch.empty((2, B, L, J), device=G.DEV)
    g, th, hw = torch.full((J,), 0.9, device=G.DEV), torch.ones(J, device=G.DEV), torch.ones((2, H, 3), device=G.DEV)
    K.cawn_set_spin_limit(0)
    try:
        if hconv:
            st = K.cawn_phase_accumulate_hconv_fwd(d, x[0], x[1], None, None, None, g, th, None, None, hw, None, None, z[0], z[1],
                                                   None, None, None, ws)
        else:
            st = K.cawn_phase_accumulate_fwd(d, x[0], x[1], g, th, None, None, None, z[0], z[1], None, None, None, ws)
        assert st == K.CAWN_OK
        status = K.cawn_workspace_status(ws)
    finally:
        K.cawn_set_spin_limit(1 << 20)
    assert status in (K.CAWN_OK, K.CAWN_ETIMEOUT)      # (a tile whose predecessors were all done never waits)
    assert int(ws[:64].abs().sum()) == 0, "tickets"    # counters of queues 0 and 1
    for again in range(2):
        _check(B, H, F, 3, hconv=hconv, seed=4 + again, L=L, ws=ws)


def _training_calls(B, L, H, F, ret, hconv=False, seed=0):
    """A forward and a backward through the C ABI, conv 3, plain or with the valve and retentions; the workspace they share and
    a function that makes one of the calls on a stream and returns what it writes."""
    G = _gpu()
    from paper_2604_04250_amd import binding as K
    import torch
    J, Kc = H * F, 3
    g = torch.Generator(device=G.DEV)
    g.manual_seed(9500 + seed)
    n = lambda *s: torch.randn(s, device=G.DEV, generator=g)
    d = K.make_desc(B, L, H, F, conv_k=Kc, gate_tau=0.0 if ret else 0.25, amp_mode=int(ret), gate_mode=int(ret), ret_mode=int(ret),
                    hconv_k=3 if hconv else 0)
    ws = torch.empty((K.cawn_workspace_bytes(d) + 3) // 4, dtype=torch.int32, device=G.DEV)
    K.check(K.cawn_workspace_init(ws))
    x, dz, cw, cb, ck = n(2, B, L, J), n(2, B, L, J), n(2, J, Kc) / 3 ** 0.5, 0.1 * n(2, J), n(K.cawn_ckpt_bytes(d) // 4)
    valve, rl, rb = (n(B, L, H) * 3 - 3.9, n(B, L, H) * 1.5 - 2, torch.linspace(3, 0, F, device=G.DEV)) if ret else (None,) * 3
    gamma = None if ret else 0.9 + 0.0999 * torch.rand(J, device=G.DEV, generator=g)
    theta, hw, hb = torch.rand(J, device=G.DEV, generator=g) * np.pi, n(2, H, 3), n(2, H)

    def fwd(stream=None):
        z = torch.full((2, B, L, J), float("nan"), device=G.DEV)
        tail = (None, z[0], z[1], None, ck, None, ws)
        if hconv:
            st = K.cawn_phase_accumulate_hconv_fwd(d, x[0], x[1], valve, rl, rb, gamma, theta, cw, cb, hw, hb, *tail, stream=stream)
        elif ret:
            st = K.cawn_phase_accumulate_ret_fwd(d, x[0], x[1], valve, rl, rb, theta, cw, cb, *tail, stream=stream)
        else:
            st = K.cawn_phase_accumulate_fwd(d, x[0], x[1], gamma, theta, cw, cb, *tail, stream=stream)
        K.check(st)
        return [z, ck]

    def bwd(stream=None):
        e = lambda *s: torch.full(s, float("nan"), device=G.DEV)
        dx, dl, par = e(2, B, L, J), [e(B, L, H), e(B, L, H)] if ret else [], [e(J), e(2, J, Kc), e(2, J)]
        dg, dh = [] if ret else [e(J)], [e(2, H, 3), e(2, H)] if hconv else []
        up = (None, ck, dz[0], dz[1], None, dx[0], dx[1])
        if hconv:
            st = K.cawn_phase_accumulate_hconv_bwd(d, x[0], x[1], valve, rl, rb, gamma, theta, cw, cb, hw, hb, *up, *(dl or (None, None)),
                                                   *(dg or (None,)), *par, *dh, None, ws, stream=stream)
        elif ret:
            st = K.cawn_phase_accumulate_ret_bwd(d, x[0], x[1], valve, rl, rb, theta, cw, cb, *up, *dl, *par, None, ws, stream=stream)
        else:
            st = K.cawn_phase_accumulate_bwd(d, x[0], x[1], gamma, theta, cw, cb, *up, *dg, *par, None, ws, stream=stream)
        K.check(st)
        return [dx] + dl + dg + par + dh
    return ws, fwd, bwd


# one tile a workgroup in both calls, on rows of 32, 64, 128 and 256 lanes in the forward; several tiles a workgroup (1071, 2079)
@pytest.mark.parametrize("B,L,H,F,hconv", [(1, 4200, 4, 32, False), (1, 2000, 4, 64, True), (2, 700, 2, 128, True), (1, 900, 2, 256, True),
                                           (21, 4200, 3, 32, False)])
@pytest.mark.parametrize("ret", [False, True])
def test_a_forward_or_backward_that_gave_up_says_so_or_is_right(B, L, H, F, hconv, ret):
    """With a spin limit of zero, set from the host, a call either reports that a wait gave up or has the results of the
    call that waits; it leaves the workspace ready in both cases."""
    from paper_2604_04250_amd import binding as K
    import torch
    ws, fwd, bwd = _training_calls(B, L, H, F, ret, hconv, seed=11)
    ref = {fwd: [t.clone() for t in fwd()], bwd: [t.clone() for t in bwd()]}
    for call in (bwd, fwd):                             # (the backward reads the checkpoints of a forward that waited)
        torch.cuda.synchronize()
        K.cawn_set_spin_limit(0)
        try:
            out = call()
            status = K.cawn_workspace_status(ws)
        finally:
            K.cawn_set_spin_limit(1 << 20)
        assert status == K.CAWN_ETIMEOUT or (status == K.CAWN_OK and all(torch.equal(a, b) for a, b in zip(ref[call], out)))
        assert int(ws[:64].abs().sum()) == 0, "tickets"    # counters of queues 0 and 1
    for call in (fwd, bwd):
        out = call()
        K.check(K.cawn_workspace_status(ws))
        assert all(torch.equal(a, b) for a, b in zip(ref[call], out))


# A workgroup for every tile, more than the chip holds at a time even alone: 960 tiles of 32 lanes, 768 with the valve and
# retentions, 1536 of 64 lanes with the harmonic convolution (256 compute units; 3, 2 and 2 of them a compute unit)
@pytest.mark.parametrize("B,L,H,F,ret,hconv", [(4, 4096, 15, 32, False, False), (4, 4096, 6, 64, True, False), (4, 4096, 12, 64, True, True)])
def test_more_tiles_than_fit_on_two_streams(B, L, H, F, ret, hconv):
    """Two forward + backward calls at the same time, a workspace each, no grid resident as a whole: results equal those of the
    same calls one after the other, bit for bit, and no wait gave up."""
    from paper_2604_04250_amd import binding as K
    import torch
    jobs = [_training_calls(B, L, H, F, ret, hconv, seed=s) for s in range(2)]
    ref = [[t.clone() for t in fwd() + bwd()] for _, fwd, bwd in jobs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]    # (default priority)
    for _ in range(3):
        got = []
        for (_, fwd, bwd), s in zip(jobs, streams):
            with torch.cuda.stream(s):                      # allocations belong to the stream
                got.append(fwd(s) + bwd(s))
        torch.cuda.synchronize()
        for (ws, _, _), r, o in zip(jobs, ref, got):
            K.check(K.cawn_workspace_status(ws))
            assert all(torch.equal(a, b) for a, b in zip(r, o))


# a workgroup for every tile in both calls, in the forward only (backward tiles are half as long: 594), in neither (1071 forward
# tiles, 2079 backward)
@pytest.mark.parametrize("B,L,H,F,hconv", [(1, 4200, 4, 32, False), (1, 4200, 4, 64, True), (6, 4200, 3, 32, False), (21, 4200, 3, 32, False)])
@pytest.mark.parametrize("ret", [False, True])
@pytest.mark.parametrize("backward_wraps", [False, True])
def test_epoch_wraps_in_a_long_forward_or_a_backward(B, L, H, F, hconv, ret, backward_wraps):
    """The call that wraps a workspace's epoch (every 2^23 - 1 calls) clears what was published: with the counter set from the host so
    that it is the forward, or the backward, this call and those after it equal those before, bit for bit."""
    from paper_2604_04250_amd import binding as K
    import torch
    ws, fwd, bwd = _training_calls(B, L, H, F, ret, hconv, seed=7)
    ref = [t.clone() for t in fwd() + bwd()]
    EPOCH_WORD, EPOCH_MOD = 64 + 2, (1 << 23) - 1     # header: 64 ticket words, finished count, error flag, epoch
    torch.cuda.synchronize()
    assert int(ws[EPOCH_WORD]) == 2
    ws[EPOCH_WORD] = EPOCH_MOD - (2 if backward_wraps else 1)
    for n in range(3):
        out = fwd() + bwd()
        torch.cuda.synchronize()
        K.check(K.cawn_workspace_status(ws))
        assert int(ws[EPOCH_WORD]) == 2 * n + (0 if backward_wraps else 1)
        assert all(torch.equal(a, b) for a, b in zip(ref, out))
