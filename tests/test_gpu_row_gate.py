"""Backward with one gate logit per (token, head) over the whole range of the
sigmoid: logits from -200 (a sigmoid of exactly 0) to 30, one head shut almost
wholly.  The gradients of every head are held to the bf16 rules relative to that
head alone, dq also per logit, on each kernel that the gated backward reaches."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_31248_amd import binding as B
from paper_2606_31248_amd import inputs as I
from _util import check_close, dev_tensor, host_f64
from test_gpu_options import check_bwd_grads, coords_for, gpu_phases

pytestmark = pytest.mark.gpu

LOGITS = np.array([-200.0, -60.0, -20.0, -3.0, 0.0, 4.0, 30.0], np.float32)


@pytest.mark.parametrize("shape,window", [
    ((1, 2, 5, 13, 12, 64), (5, 9, 9)),     # one-block dK/dV, 9-wide
    ((1, 2, 5, 13, 11, 64), (3, 7, 7)),     # one-block dK/dV
    ((2, 2, 20, 3, 5, 64), (20, 1, 1)),     # columns of two blocks
    ((1, 2, 9, 4, 5, 64), (5, 1, 1)),       # columns of one block
    ((1, 2, 5, 9, 10, 64), (3, 3, 3)),      # any window
    ((1, 2, 9, 10, 9, 128), (9, 9, 9)),     # head_dim 128
])
@pytest.mark.parametrize("qk_norm", [False, True])
def test_backward_over_the_sigmoid_range(shape, window, qk_norm):
    c32 = coords_for(shape, 103)
    q, k, v, dout = (I.gaussian(shape, 71, s, "bf16") for s in (0, 1, 2, I.STREAM_DO))
    pick = I.rng(71, I.STREAM_GATE).integers(0, len(LOGITS), shape[:-1])
    pick[:, 1] = 2  # a = 2e-9 throughout the second head
    g = I.f32_to_bf16_bits(LOGITS[pick])
    qd, kd, vd, gd, dod = (dev_tensor(a, "bf16") for a in (q, k, v, g, dout))
    scale = shape[-1] ** -0.5
    desc, opts, cs = B.desc_for(qd, window, scale), B.make_opts(qk_norm, 1e-6, gd), gpu_phases(c32, shape[-1])
    out = torch.empty_like(qd)
    lse = torch.empty(shape[:-1], dtype=torch.float32, device="cuda")
    B.strata_na3d_fwd_ex(desc, opts, qd, kd, vd, cs, out, lse)
    ws = torch.empty(B.strata_na3d_bwd_ex_workspace_size(desc, opts), dtype=torch.uint8, device="cuda")
    dq, dk, dv, dg = torch.empty_like(qd), torch.empty_like(qd), torch.empty_like(qd), torch.empty_like(gd)
    kept = lse.clone()
    B.strata_na3d_bwd_ex(desc, opts, qd, kd, vd, cs, out, dod, lse, dq, dk, dv, dg, ws)
    assert torch.equal(lse, kept)
    w = lambda a: oracle.widen(a, "bf16")
    refs = oracle.na3d_bwd(w(q), w(k), w(v), w(dout), window, scale, coords=c32, qk_norm=qk_norm, gate=w(g))
    if window[1] == 1 and not qk_norm:
        # D_i = <dO_i, out_i> is that of the output as it is stored in bf16; with few keys to a window its rounding
        # shows in dq and dk (2.2% and 2.7% of their RMS).  The exact results for that output differ by
        # scale d_i sum_j P_ij k_j (the forward on v = k) and scale sum_i P_ij d_i q_i (dv for dO = d q), d = D - D_stored
        # (the rotation cancels inside a column)
        ro, _ = oracle.na3d_fwd(w(q), w(k), w(v), window, scale, gate=w(g))
        d = ((ro - host_f64(out)) * w(dout)).sum(-1, keepdims=True)
        pk, _ = oracle.na3d_fwd(w(q), w(k), w(k), window, scale)
        pq = oracle.na3d_bwd(w(q), w(k), w(v), d * w(q), window, scale)[2]
        refs = (refs[0] + scale * d * pk, refs[1] + scale * pq) + tuple(refs[2:])
    for h in range(shape[1]):
        cut = lambda a: np.ascontiguousarray(a[:, h:h + 1])
        check_bwd_grads(tuple(cut(a) for a in (q, k, v, g, dout)), [t[:, h:h + 1] for t in (dq, dk, dv, dg)],
                        [cut(r) for r in refs], window, scale, "bf16", qk_norm, c32)
    got = host_f64(dq)
    for i, logit in enumerate(LOGITS):
        rows = pick == i
        if logit == -200.0:  # 1e-87: below the least bf16 value
            assert not got[rows].any()
            continue
        check_close(got[rows], refs[0][rows], "bf16", f"dq at logit {logit}")


def fits_flags(ws, shape):
    """The words of the workspace that say which (batch, head)s the balanced dK/dV pass took: they follow lse' and a
    word per row where the second term of dA would be (behind D, the dO exponents and the first term)."""
    b, h, z, y, x, d = shape
    n = b * h * z * y * x
    al = lambda m: (m + 255) // 256 * 256
    at = al(4 * n) + al(4 * b * h) + al(2 * d * n) + 8 * n
    return ws[at:at + 4 * b * h].view(torch.int32).cpu().numpy().reshape(b, h)


# 56 heads, four workgroups to each: the balanced pass fills the chip
@pytest.mark.parametrize("shape,window,kinds,norm", [((1, 56, 5, 9, 16, 64), (5, 9, 9), 4, True), ((1, 56, 9, 9, 16, 64), (9, 9, 9), 2, False)])
def test_ranges_that_float16_does_not_hold(shape, window, kinds, norm):
    """Heads by turns: ordinary; a gate open at x < 3, a = 2e-9 up to x = 7 and 1e-17 beyond (all that the keys of the
    last columns are seen by); V of 1e5; V of 1e-7 from x = 4 on.  Every four columns are held to the bf16 rule by
    themselves."""
    b, h, z, y, x, d = shape
    few = (b, kinds) + shape[2:]
    q, k, v, dout = (I.gaussian(few, 73, s, "bf16") for s in (0, 1, 2, I.STREAM_DO))
    g = I.rng(73, I.STREAM_GATE).normal(0.0, 2.0, few[:-1]).astype(np.float32)
    g[:, 1] = np.where(np.arange(x) < 3, 2.0, np.where(np.arange(x) < 8, -20.0, -39.0))
    g = I.f32_to_bf16_bits(g)
    mult = np.ones(few[:-1], np.float32)
    if kinds > 2:
        mult[:, 2] = 1e5
        mult[:, 3] = np.where(np.arange(x) < 4, 1.0, 1e-7)
    v = I.f32_to_bf16_bits(oracle.widen(v, "bf16").astype(np.float32) * mult[..., None])
    scale = d ** -0.5
    wide = [oracle.widen(a, "bf16") for a in (q, k, v, dout, g)]
    # out and lse from the oracle: the 5x9x9 forward's V has float16's range
    c32 = None if norm else coords_for(few, 104)
    ro, rl = oracle.na3d_fwd(*wide[:3], window, scale, coords=c32, qk_norm=norm, gate=wide[4])
    refs = oracle.na3d_bwd(*wide[:4], window, scale, coords=c32, qk_norm=norm, gate=wide[4])
    every = lambda a, dtype="bf16": dev_tensor(np.concatenate([a] * (h // kinds), 1), dtype)
    qd, kd, vd, dod, gd = (every(a) for a in (q, k, v, dout, g))
    out, lse = every(I.f32_to_bf16_bits(ro.astype(np.float32))), every(rl, "f32")
    desc, opts = B.desc_for(qd, window, scale), B.make_opts(norm, 1e-6, gd)
    cs = None if norm else gpu_phases(c32, d)
    ws = torch.empty(B.strata_na3d_bwd_ex_workspace_size(desc, opts), dtype=torch.uint8, device="cuda")
    dq, dk, dv, dg = torch.empty_like(qd), torch.empty_like(qd), torch.empty_like(qd), torch.empty_like(gd)
    B.strata_na3d_bwd_ex(desc, opts, qd, kd, vd, cs, out, dod, lse, dq, dk, dv, dg, ws)
    for name, t, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), refs):
        for i in range(kinds, h, kinds):
            assert torch.equal(t[:, :kinds], t[:, i:i + kinds])
        got = host_f64(t[:, :kinds])
        for i in range(kinds):
            for x0 in range(0, x, 4):
                cut = np.s_[:, i, :, :, x0:x0 + 4]
                check_close(got[cut], ref[cut], "bf16", f"{name}, head {i}, columns from {x0}")
    # the balanced pass took the ordinary heads alone
    assert np.array_equal(fits_flags(ws, shape), [[1, 0, 0, 0][:kinds] * (h // kinds)])
