"""First-layer kernels over extents of any parity and alignment, one and four
input channels, against the oracle: the fused forward (pooled output and slope
mask), the fused backward weights, non-finite inputs, and the fp32
four-channel forward against the generic kernel bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_1808_04728_amd import binding as B
from tests._util import TOL, dev, maxabs_err, tdtype, to_np

pytestmark = pytest.mark.gpu

# N, (D,H,W), pad, alpha: widths around a tile (32, 64, 128), odd rows, incomplete pairs, the smallest extents
CASES = [
    (1, (8, 9, 33), "same", 0.01),
    (2, (7, 8, 67), "valid", 0.2),     # out (5, 6, 65)
    (1, (5, 11, 131), "same", 0.01),   # three voxels past a 128-wide tile
    (1, (6, 17, 63), "same", 0.01),
    (3, (4, 4, 9), "valid", 0.01),     # out (2, 2, 7)
    (1, (9, 10, 130), "valid", 0.01),  # out (7, 8, 128), input rows of 260 bytes
    (2, (2, 2, 8), "same", 1.5),
    (1, (13, 26, 66), "same", 0.01),
]


def name(c):
    return "n%d_%dx%dx%d_%s_a%g" % (c[0], *c[1], c[2], c[3])


def unpack(mask, u):
    return np.unpackbits(mask.cpu().numpy(), bitorder="little")[:u.size].astype(bool).reshape(u.shape)


def forward(case, ci, dt, spoil=()):
    N, dhw, pad, alpha = case
    desc = B.make_desc(N, dhw, ci, 16, 3, 1, pad, dt)
    assert B.cf_conv3d_fused_supported(desc) & B.FUSED_FWD
    rng = np.random.default_rng(31)
    xs = np.log1p(rng.poisson(np.exp(rng.standard_normal((N, *dhw, ci)))))  # many exact zeros
    for at, v in spoil:
        xs[at] = v
    x = dev(xs, dt)
    w = dev(rng.standard_normal((3, 3, 3, ci, 16)) * np.sqrt(2.0 / (27 * ci)), dt)
    b = torch.as_tensor(rng.standard_normal(16) * 0.1, dtype=torch.float32, device="cuda")
    od = B.cf_conv3d_out_shape(desc)
    out = torch.full((N, *(t // 2 for t in od), 16), float("nan"), dtype=tdtype(dt), device="cuda")
    # two guard words past the mask must stay as they are
    nb = B.cf_conv3d_mask_bytes(desc)
    mask = torch.full((nb + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    B.cf_conv3d_fwd_fused(desc, x, w, b, alpha, B.CF_FUSE_POOL2, out, mask)
    torch.cuda.synchronize()
    assert bool((mask[nb:] == 0xA5).all())
    z = oracle.conv3d_fwd(to_np(x), to_np(w), pad=pad)
    return out, mask, z, to_np(b), alpha


@pytest.mark.parametrize("ci,dt", [(1, "bf16"), (4, "bf16"), (1, "f32")])
@pytest.mark.parametrize("case", CASES, ids=name)
def test_forward(case, ci, dt):
    out, mask, z, b, alpha = forward(case, ci, dt)
    u = z + b
    assert maxabs_err(to_np(out), oracle.avgpool3d_fwd(oracle.bias_lrelu_fwd(z, b, alpha))) <= TOL[dt]
    decided = np.abs(u) > 1e-5 * np.abs(u).max()
    assert np.array_equal(unpack(mask, u)[decided], (u > 0)[decided])


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("ci", [1, 4])
@pytest.mark.parametrize("case", [CASES[0], CASES[4], (1, (6, 7, 65), "same", 0.2)], ids=name)
def test_forward_non_finite(case, ci, value):
    """An infinity or NaN spoils the outputs whose window holds it and no other."""
    dhw = case[1]
    spoil = [((0, 1, 2, 4, ci - 1), value), ((0, dhw[0] - 1, 0, dhw[2] - 1, 0), value)]
    out, mask, z, b, alpha = forward(case, ci, "bf16", spoil)
    with np.errstate(invalid="ignore"):
        u = z + b
        p = oracle.avgpool3d_fwd(np.where(u > 0, u, alpha * u))
        got = to_np(out)
        fin = np.isfinite(p)
        assert np.array_equal(np.isfinite(got), fin)
        assert maxabs_err(got[fin], p[fin]) <= TOL["bf16"]
        sure = np.isfinite(u) & (np.abs(u) > 1e-5 * np.abs(u[np.isfinite(u)]).max())
        assert np.array_equal(unpack(mask, u)[sure], (u > 0)[sure])


@pytest.mark.parametrize("ci,dt", [(1, "bf16"), (4, "bf16"), (1, "f32")])
@pytest.mark.parametrize("case", CASES, ids=name)
def test_backward_weights(case, ci, dt):
    N, dhw, pad, alpha = case
    desc = B.make_desc(N, dhw, ci, 16, 3, 1, pad, dt)
    assert B.cf_conv3d_fused_supported(desc) & B.FUSED_BWD_WEIGHT
    rng = np.random.default_rng(32)
    od = B.cf_conv3d_out_shape(desc)
    x = dev(rng.standard_normal((N, *dhw, ci)), dt)
    g = dev(rng.standard_normal((N, *(t // 2 for t in od), 16)), dt)
    bits = rng.integers(0, 2, (N, *od, 16)).astype(np.uint8)
    mb = np.zeros(B.cf_conv3d_mask_bytes(desc), np.uint8)
    packed = np.packbits(bits.reshape(-1), bitorder="little")
    mb[:packed.size] = packed
    mask = torch.as_tensor(mb, device="cuda")
    dw = torch.full((3, 3, 3, ci, 16), float("nan"), device="cuda")
    db = torch.full((16,), float("nan"), device="cuda")
    ws = torch.empty(max(16, B.cf_conv3d_bwd_weight_fused_workspace_size(desc)), dtype=torch.uint8, device="cuda")
    B.cf_conv3d_bwd_weight_fused(desc, x, g, mask, alpha, B.CF_FUSE_POOL2, dw, db, ws)
    torch.cuda.synchronize()
    dy = oracle.avgpool3d_bwd(to_np(g), od)
    dz = dy * np.where(bits.astype(bool), 1.0, alpha)
    # bf16: dz may be rounded once before the product (2^-9 each, over a random sum)
    tol = 5e-3 if dt == "bf16" else TOL["f32"]
    assert maxabs_err(to_np(dw), oracle.conv3d_bwd_weight(to_np(x), dz, 3, pad=pad)) <= tol
    assert maxabs_err(to_np(db), dz.sum(axis=(0, 1, 2, 3))) <= 1e-5


@pytest.mark.parametrize("pad", ["same", "valid"])
@pytest.mark.parametrize("dhw", [(5, 9, 31), (4, 8, 32), (7, 17, 67), (3, 3, 3)])
def test_four_channel_fp32_forward_bits(dhw, pad, monkeypatch):
    """The plain fp32 forward adds the taps in the generic kernel's order."""
    desc = B.make_desc(2, dhw, 4, 16, 3, 1, pad, "f32")
    rng = np.random.default_rng(33)
    x = dev(rng.standard_normal((2, *dhw, 4)), "f32")
    w = dev(rng.standard_normal((3, 3, 3, 4, 16)), "f32")
    od = B.cf_conv3d_out_shape(desc)
    z = [torch.full((2, *od, 16), float("nan"), device="cuda") for _ in range(2)]
    B.cf_conv3d_fwd(desc, x, w, z[0])
    monkeypatch.setenv("CF_CONV_KERNEL", "igemm")
    B.cf_conv3d_fwd(desc, x, w, z[1])
    torch.cuda.synchronize()
    assert torch.equal(z[0], z[1])
    assert maxabs_err(to_np(z[0]), oracle.conv3d_fwd(to_np(x), to_np(w), pad=pad)) <= TOL["f32"]


@pytest.mark.parametrize("dhw,pad,k", [((7, 9, 33), "same", 3), ((5, 8, 67), "valid", 3), ((6, 5, 13), "same", 2),
                                       ((4, 4, 9), "valid", 3), ((3, 6, 8), "same", 3)])
def test_plain_backward_weights_one_channel(dhw, pad, k):
    """The unfused bf16 kernel (dz from memory) over the same kinds of rows."""
    desc = B.make_desc(2, dhw, 1, 16, k, 1, pad, "bf16")
    od = B.cf_conv3d_out_shape(desc)
    rng = np.random.default_rng(34)
    x = dev(rng.standard_normal((2, *dhw, 1)), "bf16")
    dz = dev(rng.standard_normal((2, *od, 16)), "bf16")
    dw = torch.full((k, k, k, 1, 16), float("nan"), device="cuda")
    ws = torch.empty(max(16, B.cf_conv3d_bwd_weight_workspace_size(desc)), dtype=torch.uint8, device="cuda")
    B.cf_conv3d_bwd_weight(desc, x, dz, dw, ws)
    torch.cuda.synchronize()
    # exact products, fp32 sums of a few thousand terms
    assert maxabs_err(to_np(dw), oracle.conv3d_bwd_weight(to_np(x), to_np(dz), k, pad=pad)) <= 1e-5


def gradient(case, ci, dt, spoil_x=(), spoil_g=(), keep=0.5):
    """The fused backward weights of a positive input, with the oracle's dz."""
    N, dhw, pad, alpha = case
    desc = B.make_desc(N, dhw, ci, 16, 3, 1, pad, dt)
    rng = np.random.default_rng(35)
    od = B.cf_conv3d_out_shape(desc)
    xs = 0.1 + np.abs(rng.standard_normal((N, *dhw, ci)))
    gs = 0.1 + np.abs(rng.standard_normal((N, *(t // 2 for t in od), 16)))
    for at, v in spoil_x:
        xs[at] = v
    for at, v in spoil_g:
        gs[at] = v
    x, g = dev(xs, dt), dev(gs, dt)
    bits = (rng.random((N, *od, 16)) < keep).astype(np.uint8)
    mb = np.zeros(B.cf_conv3d_mask_bytes(desc), np.uint8)
    packed = np.packbits(bits.reshape(-1), bitorder="little")
    mb[:packed.size] = packed
    nws = max(16, B.cf_conv3d_bwd_weight_fused_workspace_size(desc))
    # 64 guard bytes on both sides of every output and of the workspace
    bufs = [torch.full((n + 128,), 0xA5, dtype=torch.uint8, device="cuda") for n in (27 * ci * 64, 64, nws)]
    dw, db, ws = bufs[0][64:-64].view(torch.float32).view(3, 3, 3, ci, 16), bufs[1][64:-64].view(torch.float32), bufs[2][64:-64]
    B.cf_conv3d_bwd_weight_fused(desc, x, g, torch.as_tensor(mb, device="cuda"), alpha, B.CF_FUSE_POOL2, dw, db, ws)
    torch.cuda.synchronize()
    for t in bufs:
        assert bool((t[:64] == 0xA5).all()) and bool((t[-64:] == 0xA5).all())
    with np.errstate(invalid="ignore"):
        dz = oracle.avgpool3d_bwd(to_np(g), od) * np.where(bits.astype(bool), 1.0, alpha)
        return to_np(dw), to_np(db), oracle.conv3d_bwd_weight(to_np(x), dz, 3, pad=pad), dz.sum(axis=(0, 1, 2, 3))


def same_class(got, ref, tol):
    """NaN and the infinities where the reference has them, the rest within tol of its largest."""
    inf, fin = np.isinf(ref), np.isfinite(ref)
    nan_alike = np.array_equal(np.isnan(got), np.isnan(ref))
    inf_alike = np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], ref[inf])
    assert nan_alike and inf_alike
    assert maxabs_err(got[fin], ref[fin]) <= tol


@pytest.mark.parametrize("alpha", [0.0, 0.01, 1.0, 3.0])
@pytest.mark.parametrize("ci,dt,w", [(1, "bf16", 33), (1, "bf16", 40), (4, "bf16", 33), (1, "f32", 33), (1, "f32", 40)])
def test_backward_weights_infinite_gradient(ci, dt, w, alpha):
    """An infinite pooled gradient inside the volume: its channel's sums are
    infinite (NaN where the slope alpha = 0 meets it), every other sum is as
    without it."""
    for keep in (1.0, 0.5):
        spoil = [((0, 1, 1, 2, 3), np.inf), ((0, 1, 2, 9, 7), -np.inf)]
        dw, db, rw, rb = gradient((1, (6, 8, w), "same", alpha), ci, dt, spoil_g=spoil, keep=keep)
        assert np.isinf(rb[3]) or alpha == 0.0
        same_class(dw, rw, 5e-3 if dt == "bf16" else TOL["f32"])
        same_class(db, rb, 1e-5)


@pytest.mark.parametrize("alpha", [0.01, 3.0])
@pytest.mark.parametrize("ci,dt,w", [(1, "bf16", 33), (4, "bf16", 33), (1, "f32", 33)])
def test_backward_weights_infinite_input(ci, dt, w, alpha):
    """An infinite input voxel whose windows all lie in the pooled volume."""
    dw, db, rw, rb = gradient((1, (6, 8, w), "same", alpha), ci, dt, spoil_x=[((0, 2, 3, 7, ci - 1), np.inf)])
    assert np.isinf(rw[:, :, :, ci - 1]).all()
    same_class(dw, rw, 5e-3 if dt == "bf16" else TOL["f32"])
    same_class(db, rb, 1e-5)


@pytest.mark.parametrize("ci,dt,w", [(1, "bf16", 33), (1, "bf16", 40), (4, "bf16", 33), (1, "f32", 33)])
def test_backward_weights_steep_slope(ci, dt, w):
    """A slope far above 1 that no voxel takes: the kept voxels' sums must not
    drown in the rounding of alpha times all."""
    dw, db, rw, rb = gradient((1, (6, 8, w), "same", 4e6), ci, dt, keep=1.0)
    same_class(dw, rw, 5e-3 if dt == "bf16" else TOL["f32"])
    same_class(db, rb, 1e-5)


@pytest.mark.parametrize("value", [np.inf, -np.inf])
def test_forward_infinity_stays_one(value):
    """Four channels, bf16: every output whose window holds an infinite voxel
    is infinite (not NaN), at each of the 27 taps."""
    desc = B.make_desc(1, (6, 9, 21), 4, 16, 3, 1, "same", "bf16")
    rng = np.random.default_rng(36)
    xs = rng.standard_normal((1, 6, 9, 21, 4))
    xs[0, 2, 4, 7, 1] = value
    x, w = dev(xs, "bf16"), dev(rng.standard_normal((3, 3, 3, 4, 16)), "bf16")
    z = torch.full((1, 6, 9, 21, 16), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.cf_conv3d_fwd(desc, x, w, z)
    b = torch.full((16,), 0.25, device="cuda")
    out = torch.full((1, 3, 4, 10, 16), float("nan"), dtype=torch.bfloat16, device="cuda")
    mask = torch.zeros(B.cf_conv3d_mask_bytes(desc), dtype=torch.uint8, device="cuda")
    B.cf_conv3d_fwd_fused(desc, x, w, b, 0.2, B.CF_FUSE_POOL2, out, mask)
    torch.cuda.synchronize()
    ref = oracle.conv3d_fwd(to_np(x), to_np(w))
    assert np.isinf(ref).sum() == 27 * 16
    same_class(to_np(z), ref, TOL["bf16"])
    with np.errstate(invalid="ignore"):
        u = ref + 0.25
        same_class(to_np(out), oracle.avgpool3d_fwd(np.where(u > 0, u, 0.2 * u)), TOL["bf16"])
    assert np.array_equal(unpack(mask, u)[np.isinf(u)], (u > 0)[np.isinf(u)])


# rows shorter than a 16-byte vector of bf16, the smallest depths and heights, odd output widths
NARROW = [
    (1, (2, 3, 3), "same", 0.01),
    (2, (3, 2, 5), "same", 0.2),
    (1, (4, 5, 5), "valid", 0.01),   # out (2, 3, 3)
    (3, (5, 4, 7), "valid", 0.01),   # out (3, 2, 5)
    (1, (3, 3, 7), "same", 1.5),
    (2, (5, 7, 4), "valid", 0.01),   # out (3, 5, 2)
    (1, (3, 9, 9), "same", 0.01),    # one voxel more than a vector
]


@pytest.mark.parametrize("ci,dt", [(1, "bf16"), (4, "bf16"), (1, "f32")])
@pytest.mark.parametrize("case", NARROW, ids=name)
def test_narrow_rows(case, ci, dt):
    out, mask, z, b, alpha = forward(case, ci, dt)
    u = z + b
    assert maxabs_err(to_np(out), oracle.avgpool3d_fwd(oracle.bias_lrelu_fwd(z, b, alpha))) <= TOL[dt]
    decided = np.abs(u) > 1e-5 * np.abs(u).max()
    assert np.array_equal(unpack(mask, u)[decided], (u > 0)[decided])
    dw, db, rw, rb = gradient(case, ci, dt)
    same_class(dw, rw, 5e-3 if dt == "bf16" else TOL["f32"])
    same_class(db, rb, 1e-5)


# both sides of the fp32 four-channel forward's rule (rows of 16 voxels, 2^15 voxels) and the halo kernel below it
@pytest.mark.parametrize("n,dhw,pad", [(1, (6, 9, 16), "same"), (1, (6, 9, 17), "same"), (1, (16, 32, 64), "same"),
                                       (1, (16, 32, 65), "same"), (2, (7, 19, 69), "valid"), (2, (3, 5, 33), "same")])
def test_four_channel_fp32_forward_rule(n, dhw, pad, monkeypatch):
    """The plain fp32 forward by its rule, by the generic and by the halo
    kernel: the same bits."""
    desc = B.make_desc(n, dhw, 4, 16, 3, 1, pad, "f32")
    rng = np.random.default_rng(37)
    x = dev(rng.standard_normal((n, *dhw, 4)), "f32")
    w = dev(rng.standard_normal((3, 3, 3, 4, 16)), "f32")
    od = B.cf_conv3d_out_shape(desc)
    z = [torch.full((n, *od, 16), float("nan"), device="cuda") for _ in range(3)]
    B.cf_conv3d_fwd(desc, x, w, z[0])
    for k, t in zip(("igemm", "c4"), z[1:]):
        monkeypatch.setenv("CF_CONV_KERNEL", k)
        B.cf_conv3d_fwd(desc, x, w, t)
    torch.cuda.synchronize()
    assert torch.equal(z[0], z[1]) and torch.equal(z[0], z[2])
    assert maxabs_err(to_np(z[0]), oracle.conv3d_fwd(to_np(x), to_np(w), pad=pad)) <= TOL["f32"]
