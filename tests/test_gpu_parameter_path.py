"""GPU parity of what surrounds the scan kernels in a training step: the lane table built from gamma and theta, and the sums
of the parameter partials over all tiles, at the sizes where their loops change: one chain of tiles, a group more or less than
the 32 of a reduction block, a batch of eight reads per group more or less.  Bar as for the other parity tests:
rms-floored relative error <= 1e-4 against the fp64 oracle."""
import numpy as np
import pytest

from oracle import cawn_oracle as O
from test_gpu_hconv_bwd import TOL, _compare, _gpu, _inputs, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chains", [1, 31, 33, 255, 257, 300])
def test_partials_of_any_number_of_chains(chains):
    B, L, H, F, Kc = chains, 6, 5, 8, 2            # a tile a row; heads inside a lane block, the last block partly empty
    d = _inputs(B, L, H, F, Kc, 8100 + chains)
    out = _gpu().run_hconv_fwd_bwd(d, B, L, H, F, conv_k=Kc, gate_tau=0.1)
    _compare(out, _oracle(B, L, H, F, Kc, d, tau=0.1), Kc)


# Both forms of the table's angle: reduced here, and beyond 2^20 radians (theta itself, or a power's multiple of it) by the
# library.  The oracle rotates by the same fp32 theta.
@pytest.mark.parametrize("scale", [1.0, 1e4, 5e5, 3e7])
def test_lane_table_angles(scale):
    B, L, H, F, Kc = 1, 300, 2, 16, 0
    d = _inputs(B, L, H, F, Kc, 8200)
    r = np.random.Generator(np.random.PCG64(8201))
    d["theta"] = (scale * r.uniform(-1, 1, H * F)).astype(np.float32)
    d["theta"][:2] = 0.0, np.float32(np.pi / 2)
    d["gamma"][:3] = 1.0, -0.9, 0.0
    G = _gpu()
    ora = O.phase_fwd(O.Cfg(B, L, H, F), d["mag"], d["ang"], d["gamma"], d["theta"])
    out = G.run_fwd(d, B, L, H, F)
    assert max(G.rel_err(out[k], ora[k]) for k in ("z_re", "z_im")) <= TOL


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_infinite_retention_keeps_its_infinity(sign):
    """gamma = +-inf, cos and sin positive, a state (1, -1) and no input: the real part is inf + inf, the imaginary one inf - inf."""
    B, L, H, F = 1, 1, 1, 32
    G = _gpu()
    J = H * F
    d = dict(mag=np.zeros((B, L, J), np.float32), ang=np.zeros((B, L, J), np.float32), gamma=np.full(J, 0.5, np.float32),
             theta=np.linspace(0.1, 1.4, J).astype(np.float32))
    d["gamma"][::3] = sign * np.inf
    state = np.stack([np.ones((B, J)), -np.ones((B, J))], 1).astype(np.float32)
    out = G.run_fwd(d, B, L, H, F, state_in=G.pack_state(state, None))
    scan, _ = G.unpack_state(out["state_out"], B, J, 0)
    assert np.all(out["z_re"][0, 0, ::3] == sign * 100.0) and np.all(scan[0, 0, ::3] == sign * np.inf)
    assert np.all(np.isnan(scan[0, 1, ::3]))
    lam = 0.5 * np.exp(1j * d["theta"].astype(np.float64)) * (1 - 1j)
    rest = np.arange(J) % 3 != 0
    assert np.allclose(scan[0, 0, rest], lam.real[rest], rtol=1e-6) and np.allclose(scan[0, 1, rest], lam.imag[rest], rtol=1e-6)
