"""GPU parity where calls with a workgroup for every tile change their ways: chains dealt to eight ticket counters (numbers of chains
around multiples of eight, one of them alone), groups of tiles whose aggregates all segments of a workgroup read (positions
around the ends of a group of 8 or 16, and beyond the tiles one group of threads reads in a round trip), on long and short
tiles and in the backward.  Bar as for the other parity tests: rms-floored relative error <= 1e-4 against the fp64 oracle."""
import numpy as np
import pytest

from oracle import cawn_oracle as O
from test_gpu_hconv import _check, _inputs

pytestmark = pytest.mark.gpu

TOL = 1e-4


def _gpu():
    import gpu_util
    return gpu_util


def _plain_inputs(B, L, J, seed, heads=1):
    r = np.random.Generator(np.random.PCG64(seed))
    n = lambda *s: r.standard_normal(s, dtype=np.float32)
    return dict(mag=n(B, L, J), ang=n(B, L, J), gamma=r.uniform(0.9, 0.9999, J).astype(np.float32),
                theta=r.uniform(0, np.pi, J).astype(np.float32), conv_w=n(2, J, 2), conv_b=0.1 * n(2, J),
                dz_re=n(B, L, J), dz_im=n(B, L, J), valve=-3.9 + 3.0 * n(B, L, heads), ret=3.0 + n(B, L, heads))


def _forward_and_backward(B, L, F, valve, ret, seed):
    G, Kc = _gpu(), 2
    d = _plain_inputs(B, L, F, seed)
    rb = np.linspace(2.0, 0.0, F).astype(np.float32)
    kw = dict(valve=d["valve"] if valve else None, ret=d["ret"] if ret else None, ret_bias=rb if ret else None)
    cfg = O.Cfg(B, L, 1, F, conv_k=Kc, gate_mode=int(valve), gate_tau=0.0 if valve else 0.1, ret_mode=int(ret))
    a = (cfg, d["mag"], d["ang"], None if ret else d["gamma"], d["theta"])
    f = O.phase_fwd(*a, conv_w=d["conv_w"], conv_b=d["conv_b"], **kw)
    out = G.run_fwd(d, B, L, 1, F, conv_k=Kc, gate_tau=0.0 if valve else 0.1, **kw)
    assert max(G.rel_err(out[k], f[k]) for k in ("z_re", "z_im")) <= TOL
    assert np.array_equal(out["mask"], G.mask_from_gate(f["gate"]))
    g = O.phase_bwd(*a, d["dz_re"], d["dz_im"], conv_w=d["conv_w"], conv_b=d["conv_b"], **kw)
    b = G.run_fwd_bwd(d, B, L, 1, F, conv_k=Kc, gate_tau=0.0 if valve else 0.1, **kw)
    names = ["dmag", "dang", "dtheta", "dconv_w", "dconv_b"] + ([] if ret else ["dgamma"]) + ["dvalve"] * valve + ["dret"] * ret
    errs = {k: G.rel_err(b[k], g[k]) for k in names}
    assert max(errs.values()) <= TOL, errs


@pytest.mark.parametrize("chains", [1, 2, 3, 7, 8, 9, 13, 17])
@pytest.mark.parametrize("L", [200, 4300])               # short tiles; long tiles (17 of 256 tokens, 34 of the backward's)
def test_chains_over_the_counters(chains, L):
    _forward_and_backward(chains, L, 32, False, False, 9100 + chains + L)


# short tiles: 8 - 33 a chain; the backward's groups of 16 end at 2048 and 4096 tokens; long tiles with one group of 16 and more
@pytest.mark.parametrize("L", [512, 1984, 2048, 2049, 2176, 4096, 4224, 4608])
@pytest.mark.parametrize("valve,ret", [(False, False), (True, False), (False, True), (True, True)])
def test_positions_in_a_group(L, valve, ret):
    _forward_and_backward(1, L, 32, valve, ret, 9200 + L)


# 64-lane rows, two aggregates a round trip (retentions behind the harmonic convolution): groups of 8 and 16 tiles of 128 tokens
@pytest.mark.parametrize("B,L", [(1, 4224), (1, 4609), (9, 1408), (9, 5000)])
@pytest.mark.parametrize("bf16", [False, True])
def test_groups_behind_the_harmonic_convolution(B, L, bf16):
    H, F, Kc = 1, 64, 2
    _check(B, L, H, F, Kc, _inputs(B, L, H, F, Kc, 9300 + L), amp_mode=1, valve=True, ret=True, bf16=bf16)


def test_results_do_not_depend_on_timing():
    """Ten runs of one call have the same bits: the association of a chain follows from the positions of its tiles."""
    G = _gpu()
    d = _plain_inputs(3, 4500, 32, 9400)
    first = G.run_fwd_bwd(d, 3, 4500, 1, 32, conv_k=2, gate_tau=0.1)
    for _ in range(9):
        again = G.run_fwd_bwd(d, 3, 4500, 1, 32, conv_k=2, gate_tau=0.1)
        assert all(np.array_equal(first[k], again[k]) for k in ("dmag", "dang", "dgamma", "dtheta", "dconv_w", "dconv_b"))
