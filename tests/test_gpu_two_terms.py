"""The float products of larger layers from two half-precision terms per operand (the AUTO route of such layers): parity
with the oracle at the edges of its tiles and arrangements, the scales, non-finite inputs, parts of a batch, and the
float route in its place where the workspace is too small."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1501_07338_amd import vcnn
from paper_1501_07338_amd.workloads import bf16_round, random_tensor
from util import assert_close, to_np

DEV = "cuda:0"
# the split itself leaves about 1e-7 of the largest element, the float accumulation of these sums less than 2e-6
TOL = 4e-6

# (n, c, h, w, k, r, s, pad_h, pad_w): at most 32 / 48 / 64 / more maps, ragged channels, planes and batches
SHAPES = [
    (3, 102, 29, 29, 8, 16, 1, 0, 0),      # at most 32 maps, few pixels
    (10, 185, 22, 13, 23, 9, 9, 0, 0),     # 32-row tiles, long contraction
    (11, 57, 33, 31, 38, 5, 7, 2, 3),      # 33..48 maps: 16-row tiles, padded
    (17, 41, 40, 37, 49, 5, 5, 2, 2),      # one map more than the 16-row tiles take
    (23, 130, 30, 30, 64, 5, 5, 2, 2),
    (7, 29, 143, 11, 142, 12, 10, 0, 0),   # several row tiles, a short last one
    (3, 26, 147, 147, 7, 1, 80, 0, 0),     # wide kernel
    (2, 174, 27, 27, 300, 5, 5, 0, 0),     # four row groups side by side
    (7, 19, 25, 42, 9, 7, 7, 3, 3),        # short runs of the kernel gradient: waves without a share of one
]


def tensors(shape, seed):
    n, c, h, w, k, r, s, ph, pw = shape
    x = np.maximum(random_tensor(seed, (n, c, h, w)), 0)
    wt = random_tensor(seed + 1, (k, c, r, s), scale=(2.0 / (c * r * s)) ** 0.5)
    b = random_tensor(seed + 2, (k,), scale=0.1)
    d = vcnn.conv_desc(n, c, h, w, k, r, s, ph, pw)
    oh, ow = vcnn.conv_out_shape(d)
    return d, x, wt, b, random_tensor(seed + 3, (n, k, oh, ow))


def run(d, x, wt, b, dy, ws_bytes=None):
    """(y, dw, db, dx) under the current route choice, each with its own workspace of the size asked for."""
    xd, wd, bd, dyd = (torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in (x, wt, b, dy))
    out = [torch.full(a.shape, float("nan"), device=DEV) for a in (dy, wt, b, x)]

    def ws(which):
        need = vcnn.conv_workspace_bytes(d, which) if ws_bytes is None else ws_bytes[which]
        return torch.empty(need, dtype=torch.uint8, device=DEV) if need else None
    vcnn.conv_fwd(d, xd, wd, bd, out[0], ws(vcnn.PASS_FWD))
    vcnn.conv_bwd_filter(d, xd, dyd, out[1], out[2], ws(vcnn.PASS_BWD_FILTER))
    vcnn.conv_bwd_data(d, wd, dyd, out[3], ws(vcnn.PASS_BWD_DATA))
    return [to_np(t) for t in out]


def float_route_bytes(d):
    vcnn.set_conv_algo(vcnn.ALGO_IMPLICIT)
    try:
        return [vcnn.conv_workspace_bytes(d, p) for p in range(3)]
    finally:
        vcnn.set_conv_algo(vcnn.ALGO_AUTO)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
def test_two_term_products_against_the_oracle(shape):
    n, c, h, w, k, r, s, ph, pw = shape
    d, x, wt, b, dy = tensors(shape, 4100)
    assert [vcnn.conv_workspace_bytes(d, p) for p in range(3)] != float_route_bytes(d)  # the two-term route is taken
    y, dw, db, dx = run(d, x, wt, b, dy)
    assert_close(y, O.conv_fwd(x, wt, b, pad=(ph, pw)), TOL, "y")
    rdw, rdb = O.conv_bwd_filter(x, dy, (r, s), pad=(ph, pw))
    assert_close(dw, rdw, TOL, "dw")
    assert_close(db, rdb, TOL, "db")
    assert_close(dx, O.conv_bwd_data(wt, dy, (h, w), pad=(ph, pw)), TOL, "dx")
    again = run(d, x, wt, b, dy)
    assert all(np.array_equal(a, e) for a, e in zip((y, dw, db, dx), again))


@pytest.mark.gpu
def test_scales_are_exact():
    """The operands are scaled by powers of two, so inputs scaled by powers of two give the same bits, scaled."""
    d, x, wt, b, dy = tensors(SHAPES[2], 4200)
    zero = np.zeros_like(b)
    base = run(d, x, wt, zero, dy)
    e_x, e_w, e_d = 2.0 ** -80, 2.0 ** 60, 2.0 ** -30
    f = np.float32
    got = run(d, x * f(e_x), wt * f(e_w), zero, dy * f(e_d))
    for a, e, scale in zip(got, base, (e_x * e_w, e_x * e_d, e_d, e_w * e_d)):
        assert np.array_equal(a.astype(np.float64), e.astype(np.float64) * scale)
    assert not np.any(run(d, x * f(0), wt, zero, dy)[0])  # an operand of zeros has no scale


@pytest.mark.gpu
def test_non_finite_elements_stay_in_their_sums():
    n, c, h, w, k, r, s, ph, pw = shape = SHAPES[3]
    d, x, wt, b, dy = tensors(shape, 4300)
    base = run(d, x, wt, b, dy)[0]
    x[1, 7, 20, 20], x[5, 0, 3, 30] = np.inf, np.nan
    y = run(d, x, wt, b, dy)[0]
    touched = np.zeros(y.shape, bool)
    touched[1, :, 18:23, 18:23] = touched[5, :, 1:6, 28:33] = True
    assert not np.any(np.isfinite(y[touched]))
    assert np.max(np.abs(y - base)[~touched]) <= 2 * TOL * np.max(np.abs(base))


@pytest.mark.gpu
def test_a_workspace_of_the_float_route_still_runs():
    d, x, wt, b, dy = tensors(SHAPES[4], 4400)
    small = float_route_bytes(d)
    assert small[0] == 0 < vcnn.conv_workspace_bytes(d, vcnn.PASS_FWD)
    for got, want in zip(run(d, x, wt, b, dy, small), run(d, x, wt, b, dy)):
        assert_close(got, want, 2 * TOL)


@pytest.mark.gpu
def test_batch_in_parts():
    """A layer whose re-laid copies exceed what a pass asks for goes through its batch in parts (a ragged last one)."""
    shape = (67, 64, 64, 64, 32, 5, 5, 2, 2)
    n, c, h, w, k, r, s, ph, pw = shape
    d, x, wt, b, dy = tensors(shape, 4500)
    small = float_route_bytes(d)
    need = [vcnn.conv_workspace_bytes(d, p) for p in range(3)]
    assert need[0] == 0 and need[1] == small[1] <= vcnn.conv_bwd_filter_noalloc_limit()
    whole = run(d, x, wt, b, dy, [256 << 20] * 3)
    parts = run(d, x, wt, b, dy, [20 << 20, need[1], 20 << 20])
    for got, want in zip(parts, whole):
        assert_close(got, want, 2 * TOL)
    for img in (0, 66):  # first and last image, whole planes
        assert_close(parts[0][img:img + 1], O.conv_fwd(x[img:img + 1], wt, b, pad=(ph, pw)), TOL, "y")
        assert_close(parts[3][img:img + 1], O.conv_bwd_data(wt, dy[img:img + 1], (h, w), pad=(ph, pw)), TOL, "dx")
    # the kernel gradient's route depends on the shape alone: the same bits whatever more a caller has
    assert np.array_equal(parts[1], whole[1]) and np.array_equal(parts[2], whole[2])


def test_the_query_asks_for_no_more_than_its_allowance():
    """No GPU needed: the workspace query of layers whose re-laid copies are large."""
    for shape in ((64, 64, 64, 64, 32, 5, 5, 2, 2), (512, 64, 64, 64, 64, 3, 3, 1, 1), (16, 38, 64, 64, 512, 16, 16, 0, 0)):
        d = vcnn.conv_desc(*shape)
        assert vcnn.conv_workspace_bytes(d, vcnn.PASS_FWD) <= 64 << 20
    d = vcnn.conv_desc(*SHAPES[2])
    assert 0 < vcnn.conv_workspace_bytes(d, vcnn.PASS_BWD_FILTER) <= vcnn.conv_bwd_filter_noalloc_limit()


# layers whose input gradient is the transposed product on fragments: ragged maps (padded steps), a kernel matrix and planes
# that end inside a tile, one channel per tile and several, rows that may and may not be folded side by side
FOLD_SHAPES = [
    (2, 46, 27, 27, 45, 9, 9, 2, 3),
    (6, 83, 14, 10, 286, 9, 9, 0, 0),
    (3, 40, 31, 33, 130, 5, 4, 0, 1),
    (4, 19, 8, 62, 262, 7, 7, 3, 3),
    (9, 60, 8, 8, 192, 5, 5, 2, 2),
]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [vcnn.F32, vcnn.BF16])
@pytest.mark.parametrize("shape", FOLD_SHAPES)
def test_input_gradient_on_fragments(shape, dtype):
    """The transposed product from fragments, folded on chip (FOLD asks for it in float; AUTO takes it in bfloat16 where a
    correlation would leave the chip idle), with and without the derivative of the activation below."""
    n, c, h, w, k, r, s, ph, pw = shape
    bf = dtype == vcnn.BF16
    d = vcnn.conv_desc(n, c, h, w, k, r, s, ph, pw, dtype=dtype)
    oh, ow = vcnn.conv_out_shape(d)
    wt = bf16_round(random_tensor(4601, (k, c, r, s), scale=(2.0 / (k * r * s)) ** 0.5))
    dy, x = bf16_round(random_tensor(4602, (n, k, oh, ow))), bf16_round(random_tensor(4603, (n, c, h, w)))
    t = torch.bfloat16 if bf else torch.float32
    wd, dyd, xd = (torch.from_numpy(a).to(DEV).to(t) for a in (wt, dy, x))
    want = O.conv_bwd_data(wt, dy, (h, w), pad=(ph, pw))
    try:
        vcnn.set_conv_algo(vcnn.ALGO_AUTO if bf else vcnn.ALGO_FOLD)
        need = vcnn.conv_workspace_bytes(d, vcnn.PASS_BWD_DATA)
        ws = torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)
        dx = torch.full((n, c, h, w), float("nan"), dtype=t, device=DEV)
        vcnn.conv_bwd_data(d, wd, dyd, dx, ws)
        # (bfloat16: one rounding of the result to eight bits)
        assert_close(to_np(dx.float()), want, 4e-3 if bf else TOL, "dx")
        vcnn.conv_bwd_data_act(d, vcnn.ACT_RELU, xd, wd, dyd, dx, ws)
        assert_close(to_np(dx.float()), np.where(x > 0, want, 0), 4e-3 if bf else TOL, "dx, ReLU below")
    finally:
        vcnn.set_conv_algo(vcnn.ALGO_AUTO)


# 1 x 1 layers on fragments: whole and ragged tiles, odd planes (rows at any dword), padded slabs, split and whole sums
POINTWISE_SHAPES = [(16, 512, 49, 49, 512), (13, 389, 53, 51, 401), (11, 250, 33, 20, 455), (7, 260, 45, 45, 300)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", POINTWISE_SHAPES)
def test_pointwise_layers_on_fragments(shape):
    n, c, h, w, k = shape
    d, x, wt, b, dy = tensors((n, c, h, w, k, 1, 1, 0, 0), 4700)
    vcnn.set_conv_algo(vcnn.ALGO_AUTO)
    assert vcnn.conv_workspace_bytes(d, vcnn.PASS_BWD_DATA) > 0  # (the float route needs none)
    y, dw, db, dx = run(d, x, wt, b, dy)
    xm, dm = x.astype(np.float64).reshape(n, c, -1), dy.astype(np.float64).reshape(n, k, -1)
    wm = wt.astype(np.float64).reshape(k, c)
    assert_close(y.reshape(n, k, -1), wm @ xm + b[:, None].astype(np.float64), TOL, "y")
    assert_close(dx.reshape(n, c, -1), wm.T @ dm, TOL, "dx")
    assert_close(dw.reshape(k, c), (dm @ xm.transpose(0, 2, 1)).sum(0), TOL, "dw")
    assert_close(db, dm.sum((0, 2)), TOL, "db")
    small = run(d, x, wt, b, dy, float_route_bytes(d))
    for got, want in zip(small, (y, dw, db, dx)):
        assert_close(got, want, 2 * TOL)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [vcnn.F32, vcnn.BF16])
def test_kernel_gradient_with_a_run_shorter_than_the_waves_shares(dtype):
    """A last run of output rows too short for every wave to get a slab, followed by the next image group in the same
    block: the waves without a share must not carry that run's fragments into the next one."""
    n, c, h, w, k, r, s = 16, 512, 57, 10, 20, 5, 5
    d = vcnn.conv_desc(n, c, h, w, k, r, s, dtype=dtype)
    x, dy = bf16_round(random_tensor(4801, (n, c, h, w))), bf16_round(random_tensor(4802, (n, k, h - 4, w - 4)))
    t = torch.bfloat16 if dtype == vcnn.BF16 else torch.float32
    xd, dyd = (torch.from_numpy(a).to(DEV).to(t) for a in (x, dy))
    dw, db = torch.full((k, c, r, s), float("nan"), device=DEV), torch.full((k,), float("nan"), device=DEV)
    ws = torch.empty(vcnn.conv_workspace_bytes(d, vcnn.PASS_BWD_FILTER), dtype=torch.uint8, device=DEV)
    vcnn.conv_bwd_filter(d, xd, dyd, dw, db, ws)
    rdw, rdb = O.conv_bwd_filter(x, dy, (r, s))
    assert_close(to_np(dw), rdw, TOL, "dw")
    assert_close(to_np(db), rdb, TOL, "db")
