"""GPU parity of the forward through the harmonic convolution with heads of 128 and 256 harmonics (a row of the tile is a whole
head of several waves), against the fp64 oracle: the edges of its 64-token tiles, every gate and retention mode, both
activation types, a carried state, calls beyond the workgroups that fit the chip, and rows that do not start on 16 bytes.
Bars as in test_gpu_hconv.py, gate masks bit-exact."""
import numpy as np
import pytest

from test_gpu_hconv import TOL, _check, _gpu, _inputs, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [128, 256])
@pytest.mark.parametrize("L", [17, 63, 64, 65, 127, 193])
@pytest.mark.parametrize("valve,ret,bf16", [(False, False, False), (True, False, False), (True, True, True)])
def test_wide_heads_tile_edges_and_modes(F, L, valve, ret, bf16):
    B, H, Kc = 2, 2, 3
    d = _inputs(B, L, H, F, Kc, 8300 + F + L)
    _check(B, L, H, F, Kc, d, amp_mode=int(valve), valve=valve, ret=ret, tau=0.0 if valve else 0.25, bf16=bf16)


@pytest.mark.parametrize("F", [128, 256])
def test_wide_heads_carry_a_state(F):
    B, L, H, Kc = 2, 130, 1, 4
    d = _inputs(B, L, H, F, Kc, 8400 + F)
    r = np.random.Generator(np.random.PCG64(8401))
    J = H * F
    _check(B, L, H, F, Kc, d, tau=0.1, concat=True,
           state=(r.standard_normal((B, 2, J)).astype(np.float32), r.standard_normal((B, Kc - 1, 2, J)).astype(np.float32)))


# more tiles than workgroups fit: several a workgroup (256 lanes: beyond 256 tiles; 128 lanes: beyond 2304 of more than 32 chains).
# Batch rows are independent: the oracle runs on two of them.
@pytest.mark.parametrize("B,L,H,F,ret", [(3, 5600, 1, 256, True), (33, 4500, 1, 128, False)])
def test_wide_heads_several_tiles_a_workgroup(B, L, H, F, ret):
    Kc, few = 2, 2
    d = _inputs(few, L, H, F, Kc, 8500 + F)
    big = {k: (np.concatenate([v[i % few:i % few + 1] for i in range(B)]) if v.shape[:2] == (few, L) else v) for k, v in d.items()}
    ora = _oracle(few, L, H, F, Kc, d, 1, False, ret, 0.6)
    G = _gpu()
    out = G.run_fwd(big, B, L, H, F, conv_k=Kc, amp_mode=1, gate_tau=0.6, ret=big["ret"] if ret else None,
                    ret_bias=d["ret_bias"] if ret else None, hconv_w=d["hconv_w"], hconv_b=d["hconv_b"])
    for i in range(few):
        assert max(G.rel_err(out["z_re"][i], ora["c_re"][i]), G.rel_err(out["z_im"][i], ora["c_im"][i])) <= TOL
    for i in range(few, B):      # (the same inputs: the same bits)
        assert np.array_equal(out["z_re"][i], out["z_re"][i % few]) and np.array_equal(out["mask"][i], out["mask"][i % few])
    assert np.array_equal(out["mask"][:few], G.mask_from_gate(ora["gate"]))


def test_wide_heads_rows_off_sixteen_bytes():
    """The inputs start four bytes into their allocation: a workgroup for every tile, whatever their number."""
    import torch

    from paper_2604_04250_amd import binding as K
    G = _gpu()
    B, L, H, F, Kc = 3, 5600, 1, 256, 1
    J = H * F
    d = _inputs(B, L, H, F, Kc, 8600)
    ds = K.make_desc(B, L, H, F, conv_k=Kc, gate_tau=0.25, hconv_k=3)
    ws = G.Workspaces.get(ds)

    def run(off):
        x = []
        for k in ("mag", "ang"):
            buf = torch.empty(B * L * J + off, device="cuda:0")
            buf[off:] = torch.from_numpy(d[k]).flatten().to("cuda:0")
            x.append(buf[off:].view(B, L, J))
        z = [torch.full((B, L, J), float("nan"), device="cuda:0") for _ in range(2)]
        K.check(K.cawn_phase_accumulate_hconv_fwd(ds, x[0], x[1], None, None, None, G.dev(d["gamma"]), G.dev(d["theta"]),
                                                  G.dev(d["conv_w"]), G.dev(d["conv_b"]), G.dev(d["hconv_w"]), G.dev(d["hconv_b"]),
                                                  None, z[0], z[1], None, None, None, ws, activations_bf16=0))
        torch.cuda.synchronize()
        K.check(K.cawn_workspace_status(ws))
        return [v.cpu().numpy() for v in z]
    a, b = run(0), run(1)
    for u, v in zip(a, b):       # (one passes a prefix on per group of tiles as the other does: the same association)
        assert np.array_equal(u, v)


@pytest.mark.parametrize("F,ret", [(128, False), (256, False), (128, True), (256, True)])
def test_wide_heads_every_wave_reports_that_it_gave_up(F, ret):
    """Each wave of a row waits for its own lanes.  A call's published words are left valid for the next call (the host sets the epoch
    back) in the first wave's lanes alone, and with a spin limit of zero, set from the host, the other waves give up unless
    their words arrive in time: the call says so, or is right."""
    import torch

    from paper_2604_04250_amd import binding as K
    G = _gpu()
    B, L, H, Kc = 2, 64 * 12, 2, 2                   # twelve tiles a chain: read a few at a time, and by all segments
    J = H * F
    d = _inputs(B, L, H, F, Kc, 8700 + F)
    ds = K.make_desc(B, L, H, F, conv_k=Kc, gate_tau=0.25, hconv_k=3, ret_mode=int(ret))
    ws = torch.empty((K.cawn_workspace_bytes(ds) + 3) // 4, dtype=torch.int32, device=G.DEV)
    K.check(K.cawn_workspace_init(ws))
    x = [G.dev(d[k]) for k in ("mag", "ang")]
    par = [None if ret else G.dev(d["gamma"])] + [G.dev(d[k]) for k in ("theta", "conv_w", "conv_b", "hconv_w", "hconv_b")]
    rl, rb = (G.dev(d["ret"]), G.dev(d["ret_bias"])) if ret else (None, None)

    def call():
        z = torch.full((2, B, L, J), float("nan"), device=G.DEV)
        K.check(K.cawn_phase_accumulate_hconv_fwd(ds, x[0], x[1], None, rl, rb, *par, None, z[0], z[1], None, None, None, ws,
                                                  activations_bf16=0))
        return z, K.cawn_workspace_status(ws)

    right, st = call()
    assert st == K.CAWN_OK
    EPOCH_WORD = 64 + 2                              # header: 64 ticket words, finished count, error flag, epoch
    w = ws.cpu().numpy().view(np.uint32)
    assert w[EPOCH_WORD] == 1
    at = np.flatnonzero(w[1::2] == np.uint32(0xFF800001))       # {value, tag} of epoch 0; the first is lane 0 of the first tile's
    assert at.size and w.size * 4 >= 8 * at[-1]
    lane = (at - at[0]) % F
    for k in at[lane >= 64]:
        w[2 * k:2 * k + 2] = 0
    w[EPOCH_WORD] = 0
    ws.copy_(torch.from_numpy(w.view(np.int32)))
    K.cawn_set_spin_limit(0)
    try:
        z, st = call()
    finally:
        K.cawn_set_spin_limit(1 << 20)
    assert st == K.CAWN_ETIMEOUT or (st == K.CAWN_OK and torch.equal(z, right))
    z, st = call()
    assert st == K.CAWN_OK and torch.equal(z, right)
