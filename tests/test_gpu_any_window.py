"""The any-window attention kernels (float32 matrix instructions) against the CPU
oracle at the sizes where their tiling can go wrong: tiles of every shape, extents
they do not divide, boxes of one chunk and of a padded last chunk, windows that
span their axis (even ones too), each number of waves per tile with and without
waves past the last grid, every head_dim.

Tolerances: float32 data 1e-5; bf16 outputs one rounding of a float32 result, that is
half a bf16 ulp of the exact value plus the same 1e-5; bf16 gradients the parity rule
(their D comes from the forward's output as it is stored)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_31248_amd import binding as B
from paper_2606_31248_amd import inputs as I
from _util import F32_ABS, bf16_half_ulp, check_close, dev_tensor, host_f64
from test_gpu_parity import gpu_phases, oracle_coords, run_bwd, run_fwd

pytestmark = pytest.mark.gpu


def close(got, ref, dtype, what):
    tol = F32_ABS + (bf16_half_ulp(ref) * (1 + 2.0 ** -8) if dtype == "bf16" else 0.0)
    worst = float(np.max(np.abs(got - ref) - tol))
    assert worst <= 0, f"{what}: {worst:.3e} beyond the tolerance"


SHAPES = [
    # (shape, window, dtype, waves that share a tile: four below 2048 tiles of all grids, two below 4096, more where
    # the workgroups' other waves would find too few grids; tests/test_any_walk_host.py holds the numbers to the rule)
    ((1, 1, 1, 1, 1, 64), (1, 1, 1), "f32", 4),       # one token
    ((1, 2, 2, 3, 5, 128), (1, 3, 5), "bf16", 4),     # box = window, one padded chunk
    ((2, 1, 3, 6, 7, 128), (3, 3, 7), "f32", 4),
    ((1, 3, 18, 2, 3, 64), (18, 1, 1), "f32", 4),     # columns, an even window that spans its axis
    ((1, 1, 33, 3, 2, 32), (9, 1, 1), "bf16", 4),     # columns beyond 32 levels
    ((1, 2, 4, 6, 8, 32), (4, 6, 8), "f32", 4),       # every token sees every token
    ((2, 2, 5, 17, 9, 64), (3, 3, 3), "bf16", 4),
    ((1, 40, 6, 17, 19, 64), (3, 5, 5), "bf16", 1),
    ((4, 16, 8, 17, 16, 32), (3, 3, 3), "f32", 1),
    ((1, 20, 6, 17, 19, 64), (3, 5, 5), "bf16", 2),
    # an odd number of grids: two waves past the last.  (bf16 with 75 keys: D = <dO, out> takes the output as it is
    # stored, off by up to 2^-9 of each value, 2^-9 / sqrt(3) |dO| |out| / sqrt(d) in all, which dq and dk carry times
    # scale P k.  |out| falls with the square root of the keys: at 27 keys that comes to 3.2% of RMS(dq) at the worst
    # of 2.4M values, on the scalar kernels as well, and the rule allows 2%.)
    ((1, 21, 6, 17, 19, 64), (3, 5, 5), "bf16", 2),
    ((1, 31, 5, 16, 15, 32), (3, 3, 3), "f32", 2),
    ((2, 15, 5, 16, 15, 128), (3, 3, 3), "f32", 2),
    ((1, 65, 5, 16, 15, 64), (3, 3, 3), "f32", 1),    # three waves past the last grid
    ((1, 43, 6, 17, 19, 32), (3, 5, 5), "bf16", 1),   # one
]


@pytest.mark.parametrize("shape,window,dtype,waves", SHAPES)
def test_forward_and_backward(shape, window, dtype, waves):
    c32 = oracle_coords(I.random_placement(shape[0], shape[3], shape[4], 97), shape[3], shape[4])
    (q, k, v), out, lse, scale = run_fwd(shape, window, dtype, 51, c32)
    wide = [oracle.widen(a, dtype) for a in (q, k, v)]
    ro, rl = oracle.na3d_fwd(*wide, window, scale, coords=c32)
    close(host_f64(out), ro, dtype, "out")
    assert np.max(np.abs(host_f64(lse) - rl)) <= 1e-5
    (q, k, v, g), grads, scale = run_bwd(shape, window, dtype, 52, c32)
    refs = oracle.na3d_bwd(*(oracle.widen(a, dtype) for a in (q, k, v, g)), window, scale, coords=c32)
    for name, got, ref in zip(("dq", "dk", "dv"), grads, refs):
        check_close(host_f64(got), ref, dtype, name)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 32)])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_values_that_are_not_finite_stay_in_their_windows(dtype, d, bad):
    """One token of each of q, k, v, dO holds inf or NaN: the results that the oracle gives as finite (their
    windows hold none of these) are the oracle's, the others are not finite."""
    shape, window = (1, 1, 5, 16, 15, d), (3, 5, 5)
    names = ("q", "k", "v", "g")
    host = {n: oracle.widen(I.gaussian(shape, 61, s, dtype), dtype) for s, n in enumerate(names)}
    at = {"q": (0, 2, 2), "k": (4, 15, 14), "v": (2, 0, 14), "g": (2, 12, 1)}
    for n in names:
        host[n][(0, 0) + at[n] + (7,)] = bad
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    qd, kd, vd, gd = (torch.from_numpy(host[n]).to(dt).cuda() for n in names)
    scale = d ** -0.5
    desc = B.desc_for(qd, window, scale)
    out = torch.empty_like(qd)
    lse = torch.empty(shape[:-1], dtype=torch.float32, device="cuda")
    B.strata_na3d_fwd(desc, qd, kd, vd, None, out, lse)
    grads = [torch.empty_like(qd) for _ in range(3)]
    ws = torch.empty(B.strata_na3d_bwd_workspace_size(desc), dtype=torch.uint8, device="cuda")
    B.strata_na3d_bwd(desc, qd, kd, vd, None, out, gd, lse, *grads, ws)
    with np.errstate(all="ignore"):
        ro, _ = oracle.na3d_fwd(*(host[n] for n in names[:3]), window, scale)
        refs = oracle.na3d_bwd(*(host[n] for n in names), window, scale)
    for name, got, ref in zip(("out", "dq", "dk", "dv"), [out] + grads, (ro,) + tuple(refs)):
        got = host_f64(got)
        fine = np.isfinite(ref)
        assert 0 < np.count_nonzero(~fine) < ref.size // 2
        assert np.array_equal(np.isfinite(got), fine), name
        check_close(got[fine], ref[fine], dtype, name)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_token_that_sees_itself_alone(dtype):
    """One score per query and a scale that is a power of two: the score less its lse is 0, the weight 1 and no sum is
    rounded, so out = v and dv = dO bit for bit."""
    shape = (1, 3, 3, 6, 17, 32)
    q, k, v, g = (I.gaussian(shape, 53, s, dtype) for s in (0, 1, 2, I.STREAM_DO))
    qd, kd, vd, gd = (dev_tensor(a, dtype) for a in (q, k, v, g))
    desc, cs = B.desc_for(qd, (1, 1, 1), 0.125), gpu_phases(oracle_coords(I.random_placement(1, 6, 17, 97), 6, 17), 32)
    out, lse = torch.empty_like(qd), torch.empty(shape[:-1], dtype=torch.float32, device="cuda")
    B.strata_na3d_fwd(desc, qd, kd, vd, cs, out, lse)
    ws = torch.empty(B.strata_na3d_bwd_workspace_size(desc), dtype=torch.uint8, device="cuda")
    dq, dk, dv = (torch.empty_like(qd) for _ in range(3))
    B.strata_na3d_bwd(desc, qd, kd, vd, cs, out, gd, lse, dq, dk, dv, ws)
    assert torch.equal(out, vd) and torch.equal(dv, gd)


# relative error (2-norm) of float32 results where every query's scores are summed, exponentiated with expf and
# accumulated by one thread or wave per query, on inputs of the same distribution
@pytest.mark.parametrize("d,window,most", [
    (64, (3, 3, 3), dict(out=2.2e-7, dq=3.1e-7, dk=3.1e-7, dv=2.8e-7)),
    (32, (3, 7, 7), dict(out=2.2e-7, dq=4.1e-7, dk=4.2e-7, dv=4.1e-7)),
    (64, (5, 9, 9), dict(out=3.0e-7, dq=5.7e-7, dk=6.0e-7, dv=5.8e-7)),
])
def test_float32_error(d, window, most):
    shape = (1, 2, 6, 14, 17, d)
    c32 = oracle_coords(I.random_placement(1, 14, 17, 97), 14, 17)
    (q, k, v), out, _, scale = run_fwd(shape, window, "f32", 54, c32)
    (q, k, v, g), grads, scale = run_bwd(shape, window, "f32", 54, c32)
    wide = [oracle.widen(a, "f32") for a in (q, k, v, g)]
    refs = (oracle.na3d_fwd(*wide[:3], window, scale, coords=c32)[0],) + tuple(oracle.na3d_bwd(*wide, window, scale, coords=c32))
    for (name, bound), got, ref in zip(most.items(), [out] + list(grads), refs):
        err = np.linalg.norm(host_f64(got) - ref) / np.linalg.norm(ref)
        assert err <= bound, f"{name}: {err:.2e}"


def test_more_workgroups_than_one_grid_dimension_holds():
    """2^26 + 2^22 grids of one token: 17.8 million workgroups of 256 threads.  Every token sees itself alone: out = v,
    lse = scale <q, k>, dv = dO."""
    shape, base = (1 << 22, 17, 1, 1, 1, 32), 1 << 12
    gen = torch.Generator(device="cuda").manual_seed(7)
    q, k, v, g = (torch.randn((base,) + shape[1:], generator=gen, device="cuda").to(torch.bfloat16).repeat((shape[0] // base,) + (1,) * 5)
                  for _ in range(4))
    desc = B.desc_for(q, (1, 1, 1), 0.25)
    out, lse = torch.empty_like(q), torch.empty(shape[:-1], dtype=torch.float32, device="cuda")
    B.strata_na3d_fwd(desc, q, k, v, None, out, lse)
    assert torch.equal(out, v)
    want = 0.25 * (q[:base].double() * k[:base].double()).sum(-1)
    assert (lse.view(-1, *want.shape).double() - want).abs().max() <= 1e-5
    ws = torch.empty(B.strata_na3d_bwd_workspace_size(desc), dtype=torch.uint8, device="cuda")
    dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(3))
    B.strata_na3d_bwd(desc, q, k, v, None, out, g, lse, dq, dk, dv, ws)
    assert torch.equal(dv, g)
    for t in (dq, dk):  # rounding of D against <dO, v>
        assert t.abs().max() <= 1e-4
