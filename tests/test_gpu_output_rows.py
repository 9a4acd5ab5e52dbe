"""GPU tests of the forward's bfloat16 output rows: whole 128-byte lines are streamed, others not, by strides and bases.  The same
call into rows of whole lines, into rows of another stride and into planes that start off a line stores the same bits, with
and without checkpoints; the first is checked against the fp64 oracle with the bar for outputs stored as bfloat16."""
import numpy as np
import pytest

from oracle import cawn_oracle as O

pytestmark = pytest.mark.gpu


# 64-lane tiles with a workgroup each, persistent, behind the harmonic convolution; rows of a head of 128; the last tile is ragged
@pytest.mark.parametrize("B,H,F,hconv", [(4, 4, 64, False), (40, 4, 64, False), (8, 2, 64, True), (3, 1, 128, True)])
@pytest.mark.parametrize("want_ckpt", [False, True])
def test_rows_of_lines_and_others(B, H, F, hconv, want_ckpt):
    import torch

    import gpu_util as G
    from paper_2604_04250_amd import binding as K
    L, J, few = 2125, H * F, 2
    r = np.random.Generator(np.random.PCG64(9500 + B))
    n = lambda *s: r.standard_normal(s, dtype=np.float32)
    mag, ang = G.bf16_exact(n(few, L, J)), G.bf16_exact(n(few, L, J))
    gamma, theta = r.uniform(0.9, 0.9999, J).astype(np.float32), r.uniform(0, np.pi, J).astype(np.float32)
    hw, hb = 0.4 * n(2, H, 3), 0.1 * n(2, H)
    f = O.phase_fwd(O.Cfg(few, L, H, F, gate_tau=0.1), mag, ang, gamma, theta)
    ora = O.harmonic_conv(f["z_re"], f["z_im"], H, F, hw, hb) if hconv else (f["z_re"], f["z_im"])
    rows = [np.tile(x, (-(-B // few), 1, 1))[:B] for x in (mag, ang)]

    def run(stride, off):
        d = K.make_desc(B, L, H, F, gate_tau=0.1, hconv_k=3 if hconv else 0)
        d.out_stride_t, d.out_stride_b = stride, L * stride
        z = []
        for _ in range(2):
            buf = torch.full((off + B * L * stride,), float("nan"), device="cuda:0", dtype=torch.bfloat16)
            z.append(buf[off:].view(B, L, stride)[:, :, :J])
        ck = torch.empty(K.cawn_ckpt_bytes(d) // 4, device="cuda:0") if want_ckpt else None
        ws = G.Workspaces.get(d)
        a = (G.dev_bf16(rows[0]), G.dev_bf16(rows[1]), None, None, None, G.dev(gamma), G.dev(theta), None, None)
        if hconv:
            K.check(K.cawn_phase_accumulate_hconv_fwd(d, *a, G.dev(hw), G.dev(hb), None, z[0], z[1], None, ck, None, ws, activations_bf16=1))
        else:
            K.check(K.cawn_phase_accumulate_bf16_fwd(d, *a, None, z[0], z[1], None, ck, None, ws))
        torch.cuda.synchronize()
        K.check(K.cawn_workspace_status(ws))
        return [G.host_bf16(v.contiguous()) for v in z]

    lines = run(J, 0)
    assert max(G.bf16_err(u[:few], v) for u, v in zip(lines, ora)) <= 1.0
    for other in (run(J + 2, 0), run(J, 2)):
        for u, v in zip(lines, other):
            assert np.array_equal(u, v)
