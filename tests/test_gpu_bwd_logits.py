"""GPU parity of the backward with valve or retention logits where its workgroups (512 on 256 compute units) take a second
tile, on both sides of the line between gradients staged a tile ahead and gradients loaded at a tile's top (launch_bwd_vkp),
against the fp64 oracle through the C ABI.  Bar as in the other parity tests; what is stored as bfloat16 may be 1e-4 off and is
then rounded."""
import numpy as np
import pytest

from oracle import cawn_oracle as O

pytestmark = pytest.mark.gpu

TOL = 1e-4


def _gpu():
    import gpu_util
    return gpu_util


def _inputs(B, L, H, F, Kc, valve, ret, hconv, bf16, seed):
    G = _gpu()
    r = np.random.Generator(np.random.PCG64(seed))
    J, kk = H * F, max(Kc, 1)
    n = lambda *s: r.standard_normal(s, dtype=np.float32)
    ex = G.bf16_exact if bf16 else (lambda x: x)
    d = dict(mag=ex(n(B, L, J)), ang=ex(n(B, L, J)), dz_re=ex(n(B, L, J)), dz_im=ex(n(B, L, J)),
             gamma=r.uniform(0.9, 0.9999, J).astype(np.float32), theta=r.uniform(0, np.pi, J).astype(np.float32),
             conv_w=n(2, J, kk) / np.float32(np.sqrt(kk)), conv_b=0.1 * n(2, J))
    d["dc_re"], d["dc_im"] = d["dz_re"], d["dz_im"]
    if hconv:
        d.update(hconv_w=n(2, H, 3), hconv_b=n(2, H))
    modes = dict(valve=-3.9 + 3.0 * n(B, L, H) if valve else None, ret=-2.0 + 1.5 * n(B, L, H) if ret else None,
                 ret_bias=np.linspace(3.0, 0.0, F, dtype=np.float32) if ret else None)
    state = [n(B, 2, J), n(B, max(Kc - 1, 0), 2, J)]
    dstate = [n(B, 2, J), n(B, max(Kc - 1, 0), 2, J)]
    return d, modes, state, dstate


def _check(B, L, H, F, Kc, valve, ret, hconv=False, bf16=False, concat=False, want_param=True, seed=0, pad=0):
    G = _gpu()
    J = H * F
    d, modes, state, dstate = _inputs(B, L, H, F, Kc, valve, ret, hconv, bf16, 8700 + seed + 131 * H + F + Kc)
    amp, tau = (1, 0.0) if valve else (0, 0.25)
    blobs = dict(state_in=G.pack_state(*state), dstate_out=G.pack_state(*dstate))
    kw = dict(conv_k=Kc, amp_mode=amp, gate_tau=tau)
    if hconv:
        out = G.run_hconv_fwd_bwd(d, B, L, H, F, bf16=bf16, concat=concat, **kw, **modes, **blobs)
    elif bf16:
        out = G.run_fwd_bwd_bf16(d, B, L, H, F, concat=concat, pad=pad, want_param=want_param, **kw, **modes, **blobs)
    else:
        out = G.run_fwd_bwd(d, B, L, H, F, concat=concat, pad=pad, want_param=want_param, **kw, **modes, **blobs)
    okw = dict(kw, gate_mode=int(valve), ret_mode=int(ret))
    st = dict(scan_in=state[0].astype(np.float64), tail_in=state[1] if Kc > 1 else None)
    streams = dict(conv_w=d["conv_w"], conv_b=d["conv_b"], **modes)
    gamma = None if ret else d["gamma"]
    dz = d["dz_re"], d["dz_im"]
    if hconv:
        f = O.phase_fwd(O.Cfg(B, L, H, F, **okw), d["mag"], d["ang"], gamma, d["theta"], **streams, **st)
        gh = O.harmonic_conv_bwd(f["z_re"], f["z_im"], H, F, d["hconv_w"], d["dc_re"], d["dc_im"])
        dz = gh["dz_re"], gh["dz_im"]
    ora = O.phase_bwd(O.Cfg(B, L, H, F, dz_f64=int(hconv), **okw), d["mag"], d["ang"], gamma, d["theta"], *dz,
                      dscan_out=dstate[0].astype(np.float64), dtail_out=dstate[1].astype(np.float64) if Kc > 1 else None,
                      **streams, **st)
    if hconv:
        ora.update(dhconv_w=gh["dw"], dhconv_b=gh["dbias"])
    names = ["dtheta", "dgamma", "dconv_w", "dconv_b", "dhconv_w", "dhconv_b", "dvalve", "dret"]
    errs = {k: G.rel_err(out[k], ora[k]) for k in names if k in out}
    assert len(errs) >= int(valve) + int(ret) + int(want_param)
    for k in ("dmag", "dang"):
        errs[k] = G.bf16_err(out[k], ora[k]) * TOL if bf16 else G.rel_err(out[k], ora[k])
    dsc, dtl = G.unpack_state(out["dstate_in"], B, J, Kc)
    errs["dscan_in"] = G.rel_err(dsc, ora["dscan_in"])
    if Kc > 1:
        errs["dtail_in"] = G.rel_err(dtl, ora["dtail_in"])
    assert max(errs.values()) <= TOL, errs


# A second tile with its gradients staged ahead: odd numbers of tokens, heads of 8 to 64, blocks of lanes not all full; chains
# beyond 64 (32 with retentions and, in fp32, behind the harmonic convolution), tiles beyond the line (1024 with the valve, 768
# with retentions, 512 with both, in bf16 2048, 2048 and 1024, behind the harmonic convolution 1024)
@pytest.mark.parametrize("B,L,H,F,Kc,valve,ret,hconv,bf16", [
    (24, 1859, 9, 8, 3, True, False, False, False), (24, 1859, 9, 8, 0, True, False, False, False),
    (11, 3101, 9, 8, 4, False, True, False, False), (11, 3101, 9, 8, 0, False, True, False, False),
    (11, 1999, 5, 16, 3, True, True, False, False), (11, 1999, 5, 16, 0, True, True, False, False),
    (24, 3700, 9, 8, 3, True, False, False, True), (11, 8001, 3, 32, 2, False, True, False, True),
    (11, 4001, 5, 16, 3, True, True, False, True), (11, 4001, 5, 16, 0, True, True, False, True),
    (6, 3700, 3, 64, 3, True, True, True, False), (11, 4101, 3, 32, 0, False, True, True, False), (12, 3700, 3, 32, 3, True, False, True, False),
    (11, 4101, 3, 32, 3, True, True, True, True), (6, 3700, 3, 64, 0, False, True, True, True), (24, 1859, 3, 32, 3, True, False, True, True)])
def test_second_tile_staged_ahead(B, L, H, F, Kc, valve, ret, hconv, bf16):
    _check(B, L, H, F, Kc, valve, ret, hconv, bf16)


def test_second_tile_staged_ahead_without_parameter_gradients():
    _check(24, 1859, 9, 8, 3, True, False, want_param=False)


# More tiles than workgroups and as many chains as the last that draw late
@pytest.mark.parametrize("B,L,H,F,valve,ret,hconv,bf16", [(16, 2300, 4, 32, True, False, False, False), (8, 5100, 4, 32, False, True, False, True),
                                                          (8, 4200, 4, 32, True, False, True, False)])
def test_second_tile_at_the_line_of_few_chains(B, L, H, F, valve, ret, hconv, bf16):
    _check(B, L, H, F, 3, valve, ret, hconv, bf16)


# ... and loaded at the tile's top: few chains of many tiles; many chains of up to two tiles a workgroup, the tail tiles with
# few tokens; and rows of J + 2 elements (4-byte staging, bfloat16 lanes at odd distances from a line)
@pytest.mark.parametrize("B,L,H,F,Kc,valve,ret,hconv,bf16,pad", [
    (4, 6000, 9, 8, 3, True, False, False, False, 0), (4, 6000, 9, 8, 0, True, False, False, True, 2),
    (3, 14800, 3, 32, 3, False, True, False, False, 2), (5, 4400, 5, 16, 0, False, True, False, True, 0),
    (5, 4800, 5, 16, 4, True, True, False, False, 0), (5, 4800, 5, 16, 3, True, True, False, True, 2),
    (1, 12000, 3, 128, 3, True, True, True, False, 0), (3, 8000, 2, 64, 3, True, False, True, True, 0), (3, 8000, 2, 64, 0, False, True, True, False, 0),
    (90, 300, 3, 16, 2, True, False, False, False, 0), (70, 389, 3, 32, 3, True, False, False, True, 2), (63, 380, 9, 8, 4, False, True, False, False, 0),
    (130, 260, 3, 16, 1, True, True, False, True, 0), (80, 257, 2, 64, 3, True, True, True, False, 0)])
def test_second_tile_loaded_at_its_top(B, L, H, F, Kc, valve, ret, hconv, bf16, pad):
    _check(B, L, H, F, Kc, valve, ret, hconv, bf16, pad=pad)


def test_loaded_at_the_top_without_parameter_gradients():
    _check(4, 6000, 9, 8, 3, True, False, want_param=False, pad=2)
    _check(1, 300, 9, 8, 3, True, False, want_param=False)
