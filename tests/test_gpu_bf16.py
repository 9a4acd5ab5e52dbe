"""GPU parity with bfloat16 activations in memory (the paper's precision split, Sec. 3.5 / Sec. 6.1:
bf16 network, fp32 accumulator) against the fp64 oracle on the same bf16-exact inputs, through the C
ABI.  Outputs stored as bf16 are allowed the rounding to nearest on top of the usual 1e-4; everything
that stays fp32 (state, checkpoints, parameter gradients) keeps the 1e-4 bar; gate masks bit-exact."""
import numpy as np
import pytest

from oracle import cawn_oracle as O

pytestmark = pytest.mark.gpu

TOL = 1e-4


def _gpu():
    import gpu_util
    return gpu_util


def _inputs(B, L, H, F, Kc, seed):
    G = _gpu()
    r = np.random.Generator(np.random.PCG64(seed))
    J = H * F
    d = dict(mag=G.bf16_exact(r.standard_normal((B, L, J), dtype=np.float32)),
             ang=G.bf16_exact(r.standard_normal((B, L, J), dtype=np.float32)),
             gamma=r.uniform(0.9, 0.999, J).astype(np.float32),
             theta=r.uniform(0, np.pi, J).astype(np.float32),
             valve=(-3.9 + 3.0 * r.standard_normal((B, L, H))).astype(np.float32),
             ret=(1.0 + 1.5 * r.standard_normal((B, L, H))).astype(np.float32),
             ret_bias=np.linspace(3.0, 0.0, F).astype(np.float32),
             dz_re=G.bf16_exact(r.standard_normal((B, L, J), dtype=np.float32)),
             dz_im=G.bf16_exact(r.standard_normal((B, L, J), dtype=np.float32)))
    kk = max(Kc, 1)
    d["conv_w"] = (r.standard_normal((2, J, kk)) / np.sqrt(kk)).astype(np.float32)
    d["conv_b"] = (0.1 * r.standard_normal((2, J))).astype(np.float32)
    return d


def _check_fwd(B, L, H, F, Kc, d, amp_mode=0, valve=False, ret=False, tau=0.0, state=None, **kw):
    G = _gpu()
    J = H * F
    scan_in = tail_in = blob = None
    if state is not None:
        scan_in, tail_in = state
        blob = G.pack_state(scan_in, tail_in if Kc > 1 else None)
    cfg = O.Cfg(B, L, H, F, conv_k=Kc, amp_mode=amp_mode, gate_mode=1 if valve else 0, gate_tau=tau,
                ret_mode=1 if ret else 0)
    ora = O.phase_fwd(cfg, d["mag"][:, :L], d["ang"][:, :L], None if ret else d["gamma"], d["theta"],
                      conv_w=d["conv_w"], conv_b=d["conv_b"], valve=d["valve"][:, :L] if valve else None,
                      ret=d["ret"][:, :L] if ret else None, ret_bias=d["ret_bias"] if ret else None,
                      scan_in=None if scan_in is None else scan_in.astype(np.float64),
                      tail_in=tail_in if Kc > 1 else None)
    out = G.run_fwd_bf16(d, B, L, H, F, conv_k=Kc, amp_mode=amp_mode, gate_tau=tau, state_in=blob,
                         valve=d["valve"] if valve else None, ret=d["ret"] if ret else None,
                         ret_bias=d["ret_bias"] if ret else None, **kw)
    e = max(G.bf16_err(out["z_re"], ora["z_re"]), G.bf16_err(out["z_im"], ora["z_im"]))
    assert e <= 1.0, e
    assert np.array_equal(out["mask"], G.mask_from_gate(ora["gate"])), "gate mask differs"
    scan, tail = G.unpack_state(out["state_out"], B, J, Kc)
    assert G.rel_err(scan, ora["scan_out"]) <= TOL               # the carried state stays fp32
    if Kc > 1:
        assert np.array_equal(tail, ora["tail_out"])
    return out, ora


def test_bf16_helpers_round_to_nearest_even():
    G = _gpu()
    x = np.array([1.0, 1.00390625, 1.01171875, -2.5, 3.0e38, 1e-40, 0.0], np.float32)
    # 1 + 2^-8 lies halfway between 1 and 1 + 2^-7: ties go to the even mantissa (1.0);
    # 1 + 3 * 2^-8 lies halfway between 1 + 2^-7 and 1 + 2^-6: the even one is 1 + 2^-6
    got = G.bf16_exact(x)
    assert got[0] == 1.0 and got[1] == 1.0 and got[2] == 1.015625 and got[3] == -2.5 and got[6] == 0.0
    assert abs(float(got[4]) / float(x[4]) - 1) <= 2.0 ** -8


@pytest.mark.parametrize("H,F", [(3, 64), (2, 32), (4, 16), (1, 128), (5, 32)])
@pytest.mark.parametrize("Kc", [0, 4])
def test_bf16_forward_head_widths(H, F, Kc):
    B, L = 2, 700                      # eleven 64-token tiles, ragged tail
    d = _inputs(B, L, H, F, Kc, 7700 + H * 131 + F + Kc)
    out, ora = _check_fwd(B, L, H, F, Kc, d, tau=0.25)
    # the outputs really are bf16 values
    G = _gpu()
    assert np.array_equal(out["z_re"], G.bf16_exact(out["z_re"]))


@pytest.mark.parametrize("valve,ret", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("Kc", [0, 3])
def test_bf16_forward_valve_and_retention(valve, ret, Kc):
    B, L, H, F = 2, 600, 3, 64
    d = _inputs(B, L, H, F, Kc, 7900 + Kc + 2 * valve + 4 * ret)
    _check_fwd(B, L, H, F, Kc, d, amp_mode=1, valve=valve, ret=ret)


@pytest.mark.parametrize("L", [1, 5, 16, 17, 255, 256, 257, 515])
def test_bf16_forward_lengths_with_carried_state(L):
    B, H, F, Kc = 3, 2, 64, 4
    d = _inputs(B, 520, H, F, Kc, 8100 + L)
    r = np.random.Generator(np.random.PCG64(8))
    state = (r.standard_normal((B, 2, H * F)).astype(np.float32),
             r.standard_normal((B, Kc - 1, 2, H * F)).astype(np.float32))
    _check_fwd(B, L, H, F, Kc, d, state=state)


def test_bf16_forward_chunked_state_and_concat_layout():
    G = _gpu()
    B, L, H, F, Kc = 2, 1000, 2, 64, 4
    J = H * F
    d = _inputs(B, L, H, F, Kc, 8200)
    one, ora = _check_fwd(B, L, H, F, Kc, d, concat=True)
    blob = None
    zs = []
    for lo, hi in ((0, 300), (300, 310), (310, 1000)):     # a long, a short (step kernel) and a long call
        part = {k: (v[:, lo:hi] if k in ("mag", "ang") else v) for k, v in d.items()}
        o = G.run_fwd_bf16(part, B, hi - lo, H, F, conv_k=Kc, state_in=blob)
        blob = o["state_out"]
        zs.append(o["z_re"])
    z = np.concatenate(zs, axis=1)
    assert G.bf16_err(z, ora["z_re"]) <= 1.0
    assert G.rel_err(G.unpack_state(blob, B, J, Kc)[0], ora["scan_out"]) <= TOL


# chains of 66 short tiles, more than short tiles are taken for: 64-lane rows.  Heads of a quarter, half, all and two of a
# row; of 96, 160 and 224, which end in the middle of one; a last row that is half empty
@pytest.mark.parametrize("H,F", [(8, 8), (5, 16), (3, 32), (3, 64), (3, 96), (4, 96), (2, 128), (2, 160), (2, 224)])
@pytest.mark.parametrize("valve,ret", [(False, False), (True, False), (False, True), (True, True)])
def test_bf16_forward_long_tiles(H, F, valve, ret):
    if valve and ret and F < 16:
        pytest.skip("heads of 8 with both logits are refused")
    B, L, Kc = 1, 4200, 3
    J = H * F
    d = _inputs(B, L, H, F, Kc, 8300 + H * 131 + F + 2 * valve + ret)
    r = np.random.Generator(np.random.PCG64(83))
    state = (r.standard_normal((B, 2, J)).astype(np.float32), r.standard_normal((B, Kc - 1, 2, J)).astype(np.float32))
    out, ora = _check_fwd(B, L, H, F, Kc, d, amp_mode=1 if valve else 0, valve=valve, ret=ret, tau=0.25, state=state,
                          want_ckpt=True)
    # a checkpoint is the unclamped state before every eighth token, and no state here reaches the clamp
    z = np.stack([ora["z_re"], ora["z_im"]], 2)
    assert np.abs(z).max() < 100.0
    before = np.concatenate([state[0][:, None].astype(np.float64), z[:, 7:L - 1:8]], 1)
    assert _gpu().rel_err(out["ckpt"].reshape(before.shape), before) <= TOL


# Either side of the lines between the kernel whose threads read their rows themselves and the one that stages them (33 tiles a
# chain, 256 compute units): 512, 768 and 1792 tiles with a constant retention, of which those from 513 to 768, a workgroup
# each, and from 1793 on, several a workgroup, are staged; 1024 with the valve, 2048 with retentions
@pytest.mark.parametrize("B,valve,ret", [(15, False, False), (16, False, False), (23, False, False), (24, False, False), (54, False, False),
                                         (55, False, False), (31, True, False), (32, True, False), (62, False, True), (63, False, True)])
def test_bf16_forward_around_the_line_between_one_and_several_a_workgroup(B, valve, ret):
    L, H, F, Kc = 4200, 1, 64, 3
    r = np.random.Generator(np.random.PCG64(84))
    state = (r.standard_normal((B, 2, F)).astype(np.float32), r.standard_normal((B, Kc - 1, 2, F)).astype(np.float32))
    _check_fwd(B, L, H, F, Kc, _inputs(B, L, H, F, Kc, 8370 + B), amp_mode=1 if valve else 0, valve=valve, ret=ret, tau=0.25, state=state)


@pytest.mark.parametrize("B", [5, 13])
@pytest.mark.parametrize("valve,ret", [(False, False), (True, True)])
def test_bf16_forward_long_tiles_more_than_fit(valve, ret, B):
    """Tiles of 128 tokens x 64 lanes, the last block of a row half full, a head ending inside the second: 825, a workgroup
    each, more than the chip holds at a time; 2145, several a workgroup."""
    L, H, F, Kc = 4200, 3, 96, 3
    _check_fwd(B, L, H, F, Kc, _inputs(B, L, H, F, Kc, 8350 + valve), amp_mode=1 if valve else 0, valve=valve, ret=ret, tau=0.25)


# the longest chains of a single lane block that go on 64-token tiles, and one token more
@pytest.mark.parametrize("ret,L", [(False, 4096), (False, 4097), (True, 3968), (True, 3969)])
def test_bf16_last_short_and_first_long_tiles(ret, L):
    _check_fwd(1, L, 1, 32, 3, _inputs(1, L, 1, 32, 3, 8400 + L), ret=ret, tau=0.25)


def test_bf16_odd_lane_count_is_refused():
    import torch
    from paper_2604_04250_amd import binding as K
    x = torch.zeros(64, device="cuda:0")
    h = torch.zeros(64, device="cuda:0", dtype=torch.bfloat16)
    d = K.make_desc(1, 32, 1, 7)
    assert K.cawn_phase_accumulate_bf16_fwd(d, h, h, None, None, None, x, x, None, None, None, h, h, None, None, None,
                                            K.alloc_workspace(d)) == K.CAWN_EUNSUPPORTED


def _check_bwd(B, L, H, F, Kc, d, amp_mode=0, valve=False, ret=False, tau=0.0, state=None, dstate=None, **kw):
    G = _gpu()
    J = H * F
    scan_in = tail_in = blob = dblob = dscan = dtail = None
    if state is not None:
        scan_in, tail_in = state
        blob = G.pack_state(scan_in, tail_in if Kc > 1 else None)
    if dstate is not None:
        dscan, dtail = dstate
        dblob = G.pack_state(dscan, dtail if Kc > 1 else None)
    cfg = O.Cfg(B, L, H, F, conv_k=Kc, amp_mode=amp_mode, gate_mode=1 if valve else 0, gate_tau=tau,
                ret_mode=1 if ret else 0)
    ora = O.phase_bwd(cfg, d["mag"][:, :L], d["ang"][:, :L], None if ret else d["gamma"], d["theta"],
                      d["dz_re"][:, :L], d["dz_im"][:, :L], conv_w=d["conv_w"], conv_b=d["conv_b"],
                      valve=d["valve"][:, :L] if valve else None, ret=d["ret"][:, :L] if ret else None,
                      ret_bias=d["ret_bias"] if ret else None,
                      scan_in=None if scan_in is None else scan_in.astype(np.float64),
                      tail_in=tail_in if Kc > 1 else None,
                      dscan_out=None if dscan is None else dscan.astype(np.float64),
                      dtail_out=None if dtail is None or Kc <= 1 else dtail.astype(np.float64))
    out = G.run_fwd_bwd_bf16(d, B, L, H, F, conv_k=Kc, amp_mode=amp_mode, gate_tau=tau, state_in=blob, dstate_out=dblob,
                             valve=d["valve"] if valve else None, ret=d["ret"] if ret else None,
                             ret_bias=d["ret_bias"] if ret else None, **kw)
    for n in ("dmag", "dang"):                       # stored as bf16
        e = G.bf16_err(out[n], ora[n])
        assert e <= 1.0, (n, e)
    for n in ("dgamma", "dtheta", "dconv_w", "dconv_b", "dvalve", "dret"):      # fp32
        if n in out:
            e = G.rel_err(out[n], ora[n])
            assert e <= TOL, (n, e)
    dsi, dti = G.unpack_state(out["dstate_in"], B, J, Kc)
    assert G.rel_err(dsi, ora["dscan_in"]) <= TOL
    if Kc > 1:
        assert G.rel_err(dti, ora["dtail_in"]) <= TOL
    return out, ora


@pytest.mark.parametrize("H,F", [(3, 64), (2, 32), (4, 16), (1, 128)])
@pytest.mark.parametrize("Kc", [0, 2, 4])
def test_bf16_backward_head_widths(H, F, Kc):
    B, L = 2, 333                      # three backward tiles, ragged tail
    d = _inputs(B, L, H, F, Kc, 8700 + H * 131 + F + Kc)
    _check_bwd(B, L, H, F, Kc, d, tau=0.25)


@pytest.mark.parametrize("valve,ret", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("Kc", [0, 3])
def test_bf16_backward_valve_and_retention(valve, ret, Kc):
    B, L, H, F = 2, 300, 3, 64
    d = _inputs(B, L, H, F, Kc, 8900 + Kc + 2 * valve + 4 * ret)
    _check_bwd(B, L, H, F, Kc, d, amp_mode=1, valve=valve, ret=ret)


@pytest.mark.parametrize("L", [1, 7, 127, 128, 129, 400])
def test_bf16_backward_lengths_with_state_and_its_gradients(L):
    B, H, F, Kc = 3, 2, 64, 4
    J = H * F
    d = _inputs(B, 400, H, F, Kc, 9100 + L)
    r = np.random.Generator(np.random.PCG64(9))
    state = (r.standard_normal((B, 2, J)).astype(np.float32), r.standard_normal((B, Kc - 1, 2, J)).astype(np.float32))
    dstate = (r.standard_normal((B, 2, J)).astype(np.float32), r.standard_normal((B, Kc - 1, 2, J)).astype(np.float32))
    _check_bwd(B, L, H, F, Kc, d, state=state, dstate=dstate)


def test_bf16_backward_without_parameter_gradients():
    B, L, H, F, Kc = 2, 400, 2, 64, 4
    d = _inputs(B, L, H, F, Kc, 9200)
    _check_bwd(B, L, H, F, Kc, d, want_param=False)


@pytest.mark.parametrize("H,F,Kc", [(2, 64, 4), (3, 32, 0), (1, 24, 2)])
def test_bf16_backward_concat_layout(H, F, Kc):
    # rows of 2 J bf16 elements shared by each activation pair and its gradients (Sec. 3.5), with state
    B, L = 2, 333
    J = H * F
    d = _inputs(B, L, H, F, Kc, 9300 + H + F + Kc)
    r = np.random.Generator(np.random.PCG64(10))
    k1 = max(Kc - 1, 0)
    state = (r.standard_normal((B, 2, J)).astype(np.float32), r.standard_normal((B, k1, 2, J)).astype(np.float32))
    _check_bwd(B, L, H, F, Kc, d, state=state, concat=True)
