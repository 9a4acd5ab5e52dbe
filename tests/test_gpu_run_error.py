"""Error of the scan state against 64 bits on lanes whose lambda rounds badly.

Between two exact powers of lambda a kernel steps by lambda rounded to fp32.  With eps the relative error of that rounding, a
token's addition is off by eps for every step of the run it joins in, so that the state at the start of a run of n tokens is
off by (n - 1) / 2 eps on average.  Calls of a constant retention that short tiles can take are computed in runs of 8: 3.5 eps,
and 8 eps leaves as much again and more for the roundings of the sums.  In runs of 32 it would be 15.5 eps and more.  The lanes are chosen so that both parts of
lambda round by 85 - 100 % of half a unit in the last place (parts of lambda in [1/2, 1): eps = 2^-25 sqrt 2 at most); their
errors point every way, but each adds up over its own lane's tokens."""
import numpy as np
import pytest

from oracle import cawn_oracle as O

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24.5


def _lanes(r, n, unit=False):
    g = r.uniform(0.995, 0.999, 200 * n).astype(np.float32)
    t = r.uniform(0.6, 0.95, 200 * n).astype(np.float32)
    if unit:
        g = np.ones_like(g)
    lam = g.astype(np.float64) * np.exp(1j * t.astype(np.float64))
    bad = np.ones(g.size, bool)
    for p in (lam.real, lam.imag):
        bad &= np.abs(p - p.astype(np.float32)) > 0.85 * 2.0 ** -25
    assert bad.sum() >= n
    return g[bad][:n], t[bad][:n]


# B, L, H, F, harmonic convolution, valve, bf16: rows of 32 lanes with 1, 12 and 24 chains, bf16 with 24, the harmonic convolution
# with 4 and heads of 128 and 256 (rows of their own width, whole calls and several tiles a workgroup)
@pytest.mark.parametrize("B,L,H,F,hc,valve,bf16", [
    (1, 3584, 1, 32, False, False, False), (1, 2304, 12, 32, False, False, False), (2, 2048, 12, 32, False, True, False),
    (1, 1920, 24, 32, False, False, True), (1, 4096, 4, 64, True, False, False), (1, 4096, 4, 64, True, True, True),
    (1, 700, 1, 128, True, False, False), (2, 700, 1, 256, True, True, False), (1, 700, 2, 128, True, False, True),
    (3, 5600, 1, 256, True, False, False)])
def test_state_error_of_runs_of_eight(B, L, H, F, hc, valve, bf16):
    r = np.random.Generator(np.random.PCG64(9100 + L + F))
    J = H * F
    d = dict(mag=r.standard_normal((B, L, J), dtype=np.float32), ang=r.standard_normal((B, L, J), dtype=np.float32))
    d["gamma"], d["theta"] = _lanes(r, J)
    v = (-3.9 + 3.0 * r.standard_normal((B, L, H))).astype(np.float32) if valve else None
    _check(B, L, H, F, hc, bf16, d, r, gate_tau=0.0 if valve else 0.25, valve=v)


# Retentions from the data, about 0.95: the state reaches 20 tokens back, the retentions' own roundings (2^-24 each at most) add to the
# sums', and the bar is the same.  Rows of 32 lanes with 24 chains, bf16 with 64, heads of 128 and 256.
@pytest.mark.parametrize("B,L,H,F,hc,valve,bf16", [
    (2, 1472, 12, 32, False, False, False), (2, 1472, 12, 32, False, True, False), (2, 832, 32, 32, False, False, True),
    (1, 700, 2, 128, True, False, False), (2, 700, 1, 256, True, True, False), (1, 700, 1, 128, True, True, True)])
def test_state_error_with_retentions_from_the_data(B, L, H, F, hc, valve, bf16):
    r = np.random.Generator(np.random.PCG64(9200 + L + F))
    J = H * F
    d = dict(mag=r.standard_normal((B, L, J), dtype=np.float32), ang=r.standard_normal((B, L, J), dtype=np.float32))
    d["theta"] = _lanes(r, J, unit=True)[1]
    v = (-3.9 + 3.0 * r.standard_normal((B, L, H))).astype(np.float32) if valve else None
    _check(B, L, H, F, hc, bf16, d, r, gate_tau=0.0 if valve else 0.25, valve=v,
           ret=(3.0 + r.standard_normal((B, L, H))).astype(np.float32), ret_bias=np.zeros(F, np.float32))


def _check(B, L, H, F, hc, bf16, d, r, **kw):
    import gpu_util as G
    J = H * F
    if bf16:
        d.update(mag=G.bf16_exact(d["mag"]), ang=G.bf16_exact(d["ang"]))
    want = dict(kw)
    kw["want_ckpt"] = True
    if hc:
        kw.update(hconv_w=r.standard_normal((2, H, 3)).astype(np.float32), hconv_b=np.zeros((2, H), np.float32), bf16=bf16)
    out = (G.run_fwd_bf16 if bf16 and not hc else G.run_fwd)(d, B, L, H, F, **kw)
    tau = want.pop("gate_tau")
    cfg = O.Cfg(B, L, H, F, gate_mode=int(want["valve"] is not None), gate_tau=tau, ret_mode=int("ret" in want))
    ora = O.phase_fwd(cfg, d["mag"], d["ang"], d.get("gamma"), d["theta"], **want)
    nT = -(-L // 8)
    ck = out["ckpt"].reshape(B, nT, 2, J)[:, 1:].astype(np.float64)        # the states before tokens 8, 16, ...
    for p, z in enumerate((ora["z_re"], ora["z_im"])):
        want = np.asarray(z, np.float64)[:, 7:8 * (nT - 1):8]
        assert np.abs(want).max() < 100.0                                  # (the oracle's planes are clamped there)
        err = np.sqrt(np.mean((ck[:, :, p] - want) ** 2) / np.mean(want ** 2))
        assert err <= 8 * EPS, err / EPS
