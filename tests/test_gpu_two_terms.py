"""The float products of larger layers from two half-precision terms per operand (the AUTO route of such layers): parity
with the oracle at the edges of its tiles and arrangements, the scales, operands the terms do not carry (magnitudes too far
apart, infinities and NaN), parts of a batch, and the float route in its place where the workspace is too small."""
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
FWD, FILTER, DATA = vcnn.PASS_FWD, vcnn.PASS_BWD_FILTER, vcnn.PASS_BWD_DATA
IMPLICIT, FOLD, POINTWISE = "two_term", "two_term_fold", "two_term_pointwise"

# (n, c, h, w, k, r, s, pad_h, pad_w) and the passes that take a two-term route, which the test asserts one by one: at most
# 32 / 48 / 64 / 128 / more maps on the rows, ragged channels, planes and batches, either order of the fold's adds
SHAPES = [
    ((3, 102, 29, 29, 8, 16, 1, 0, 0), {FWD: IMPLICIT}),                 # at most 32 maps, few pixels
    ((10, 185, 22, 13, 23, 9, 9, 0, 0), {FWD: IMPLICIT, DATA: IMPLICIT}),  # 32-row tiles; 185 maps of an input gradient
    ((11, 57, 33, 31, 38, 5, 7, 2, 3), {FWD: IMPLICIT, DATA: IMPLICIT}),   # 33..48 maps: 16-row tiles, padded
    ((17, 41, 40, 37, 49, 5, 5, 2, 2), {FWD: IMPLICIT, DATA: IMPLICIT}),   # one map more than the 16-row tiles take
    ((23, 130, 30, 30, 64, 5, 5, 2, 2), {FWD: IMPLICIT, FILTER: IMPLICIT, DATA: IMPLICIT}),
    ((2, 89, 12, 33, 61, 9, 2, 2, 0), {FWD: IMPLICIT, DATA: IMPLICIT}),    # 65..128 rows in the input gradient
    ((7, 29, 143, 11, 142, 12, 10, 0, 0), {FWD: IMPLICIT}),              # several row tiles, a short last one
    ((2, 6, 36, 46, 244, 3, 4, 0, 0), {FILTER: IMPLICIT}),
    ((3, 26, 147, 147, 7, 1, 80, 0, 0), {FWD: IMPLICIT}),                # wide kernel
    ((2, 174, 27, 27, 300, 5, 5, 0, 0), {FWD: IMPLICIT}),                # four row groups side by side
    ((7, 19, 25, 42, 9, 7, 7, 3, 3), {FILTER: IMPLICIT}),                # short runs: waves without a share of one
    ((9, 120, 62, 23, 5, 10, 3, 0, 0), {FILTER: IMPLICIT}),              # a last run shorter than the waves' shares
    ((4, 6, 41, 51, 36, 3, 14, 0, 0), {FILTER: IMPLICIT}),               # six channels: most of a group padding
    ((5, 5, 19, 47, 59, 10, 9, 0, 0), {FILTER: IMPLICIT}),
    ((2, 46, 27, 27, 45, 9, 9, 2, 3), {FWD: IMPLICIT, FILTER: IMPLICIT, DATA: FOLD}),
    ((2, 29, 30, 6, 100, 14, 4, 3, 2), {DATA: FOLD}),                    # rows 32 apart meet: added one after the other
    ((3, 49, 10, 16, 140, 3, 14, 1, 7), {DATA: FOLD}),                   # ... several channels per tile, ragged maps
    ((2, 62, 11, 24, 99, 4, 7, 2, 3), {DATA: FOLD}),
    ((5, 339, 7, 9, 303, 2, 3, 1, 0), {DATA: FOLD}),
    ((13, 389, 53, 51, 401, 1, 1, 0, 0), {FWD: POINTWISE, DATA: POINTWISE}),  # odd planes: rows at any dword; ragged tiles
    ((11, 250, 33, 20, 455, 1, 1, 0, 0), {FWD: POINTWISE, DATA: POINTWISE}),
    ((2, 395, 12, 33, 191, 1, 1, 0, 0), {FWD: POINTWISE}),
    ((13, 512, 47, 51, 512, 1, 1, 0, 0), {FWD: POINTWISE, FILTER: POINTWISE, DATA: POINTWISE}),  # split sums, padded slabs
]
# one small layer of every pair of route and pass
ONE_EACH = [((11, 57, 33, 31, 38, 5, 7, 2, 3), FWD, IMPLICIT), ((2, 89, 12, 33, 61, 9, 2, 2, 0), DATA, IMPLICIT),
            ((7, 19, 25, 42, 9, 7, 7, 3, 3), FILTER, IMPLICIT), ((9, 120, 62, 23, 5, 10, 3, 0, 0), FILTER, IMPLICIT),
            ((2, 29, 30, 6, 100, 14, 4, 3, 2), DATA, FOLD), ((2, 62, 11, 24, 99, 4, 7, 2, 3), DATA, FOLD),
            ((2, 395, 12, 33, 191, 1, 1, 0, 0), FWD, POINTWISE), ((11, 250, 33, 20, 455, 1, 1, 0, 0), DATA, POINTWISE),
            ((13, 512, 47, 51, 512, 1, 1, 0, 0), FILTER, POINTWISE)]


def tensors(shape, seed):
    n, c, h, w, k, r, s, ph, pw = shape
    x = np.maximum(random_tensor(seed, (n, c, h, w)), 0)
    wt = random_tensor(seed + 1, (k, c, r, s), scale=(2.0 / (c * r * s)) ** 0.5)
    b = random_tensor(seed + 2, (k,), scale=0.1)
    d = vcnn.conv_desc(n, c, h, w, k, r, s, ph, pw)
    oh, ow = vcnn.conv_out_shape(d)
    return d, x, wt, b, random_tensor(seed + 3, (n, k, oh, ow))


def route(d, which):
    return vcnn.conv_route(d, which, vcnn.conv_workspace_bytes(d, which))


def run_pass(d, which, x, wt, b, dy, nbytes=None):
    """The pass's result (kernel gradient: dw and db) with a workspace of exactly the size asked for, filled with NaN."""
    xd, wd, bd, dyd = (torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in (x, wt, b, dy))
    nbytes = vcnn.conv_workspace_bytes(d, which) if nbytes is None else nbytes
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device=DEV) if nbytes else None
    out = torch.full({FWD: dy, FILTER: wt, DATA: x}[which].shape, float("nan"), device=DEV)
    if which == FWD:
        vcnn.conv_fwd(d, xd, wd, bd, out, ws)
    elif which == DATA:
        vcnn.conv_bwd_data(d, wd, dyd, out, ws)
    else:
        db = torch.full(b.shape, float("nan"), device=DEV)
        vcnn.conv_bwd_filter(d, xd, dyd, out, db, ws)
        return to_np(out), to_np(db)
    return to_np(out)


def product(d, which, x, wt, b, dy, nbytes=None):
    got = run_pass(d, which, x, wt, b, dy, nbytes)
    return got[0] if which == FILTER else got


def expected(d, which, x, wt, b, dy):
    pad = (d.pad_h, d.pad_w)
    if d.r == d.s == 1:  # (a plain product, quicker without the oracle's loops)
        xm, dm = x.astype(np.float64).reshape(d.n, d.c, -1), dy.astype(np.float64).reshape(d.n, d.k, -1)
        wm = wt.astype(np.float64).reshape(d.k, d.c)
        return {FWD: lambda: (wm @ xm + b[:, None].astype(np.float64)).reshape(dy.shape),
                DATA: lambda: (wm.T @ dm).reshape(x.shape),
                FILTER: lambda: sum(p @ q.T for p, q in zip(dm, xm)).reshape(wt.shape)}[which]()
    if which == FWD:
        return O.conv_fwd(x, wt, b, pad=pad)
    return O.conv_bwd_data(wt, dy, (d.h, d.w), pad=pad) if which == DATA else O.conv_bwd_filter(x, dy, (d.r, d.s), pad=pad)[0]


def float_bytes(d, which):
    """What the float route of the pass needs: the least workspace it runs with."""
    low, high = -1, vcnn.conv_workspace_bytes(d, which)
    while high - low > 1:
        mid = (low + high) // 2
        try:
            vcnn.conv_route(d, which, mid)
            high = mid
        except vcnn.VcnnError as e:
            assert e.status == vcnn.ERR_WORKSPACE
            low = mid
    return high


@pytest.mark.parametrize("shape", [(3, 410, 27, 27, 187, 13, 12, 0, 0), (6, 61, 27, 27, 461, 16, 16, 0, 0),
                                   (15, 314, 8, 12, 15, 9, 9, 4, 4), (20, 233, 8, 8, 325, 9, 9, 4, 4)])
def test_kernel_gradients_that_round_less_in_float_stay_there(shape):
    """No GPU needed: short sums, and planes that are mostly border, where the two-term kernel measured up to 1.5 of the float
    kernel's error against 64 bits."""
    assert route(vcnn.conv_desc(*shape), FILTER) == "implicit"


def test_sums_that_mostly_meet_the_border_stay_in_float():
    """No GPU needed: an input gradient whose 330 terms meet the zero border but for twenty, where the split alone leaves 1.5
    times the float kernel's error; the same kernel on a wider plane takes the terms."""
    assert route(vcnn.conv_desc(101, 235, 34, 34, 10, 1, 33), DATA) == "implicit"
    assert route(vcnn.conv_desc(101, 235, 34, 120, 10, 1, 33), DATA) == IMPLICIT


@pytest.mark.parametrize("shape,routes", SHAPES)
def test_routes_of_the_tested_layers(shape, routes):
    """No GPU needed: each pass below really is planned as a two-term product."""
    d = vcnn.conv_desc(*shape)
    for which, name in routes.items():
        assert route(d, which) == name, (shape, which)
    with pytest.raises(vcnn.VcnnError) as e:
        vcnn.conv_route(d, 7, 0)
    assert e.value.status == vcnn.ERR_UNSUPPORTED


@pytest.mark.gpu
@pytest.mark.parametrize("shape,routes", SHAPES)
def test_two_term_products_against_the_oracle(shape, routes):
    d, x, wt, b, dy = tensors(shape, 4100)
    for which, name in routes.items():
        assert route(d, which) == name
        got = run_pass(d, which, x, wt, b, dy)
        want = expected(d, which, x, wt, b, dy)
        if which == FILTER:
            assert_close(got[0], want, TOL, "dw")
            assert_close(got[1], dy.astype(np.float64).sum((0, 2, 3)), TOL, "db")
        else:
            assert_close(got, want, TOL, "y" if which == FWD else "dx")
        again = run_pass(d, which, x, wt, b, dy)
        assert all(np.array_equal(p, q) for p, q in zip(got, again))


@pytest.mark.gpu
@pytest.mark.parametrize("shape,which,name", ONE_EACH)
def test_scales_are_exact(shape, which, name):
    """The operands are scaled by powers of two, so inputs scaled by powers of two give the same bits, scaled."""
    d, x, wt, b, dy = tensors(shape, 4200)
    assert route(d, which) == name
    zero = np.zeros_like(b)
    base = product(d, which, x, wt, zero, dy).astype(np.float64)
    f = np.float32
    e_x, e_w, e_d = 2.0 ** -80, 2.0 ** 60, 2.0 ** -5
    got = product(d, which, x * f(e_x), wt * f(e_w), zero, dy * f(e_d))
    assert np.array_equal(got.astype(np.float64), base * {FWD: e_x * e_w, FILTER: e_x * e_d, DATA: e_w * e_d}[which])
    # an operand of zeros has no scale
    assert not np.any(product(d, which, x * f(0), wt, zero, dy * f(0)))


@pytest.mark.gpu
@pytest.mark.parametrize("shape,which,name", ONE_EACH)
def test_denormal_operand(shape, which, name):
    """An operand whose largest element is a denormal (few bits each, but exactly what the terms hold)."""
    d, x, wt, b, dy = tensors(shape, 4250)
    assert route(d, which) == name
    tiny, big = np.float32(2.0 ** -134), np.float32(2.0 ** 90)
    x, wt = (x * tiny, wt * big) if which != DATA else (x, wt * tiny)
    dy = dy * big if which != FWD else dy
    b = np.zeros_like(b)
    assert_close(product(d, which, x, wt, b, dy), expected(d, which, x, wt, b, dy), TOL)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,which,name", [t for t in ONE_EACH if t[1] != FILTER])
def test_an_image_does_not_depend_on_its_neighbours(shape, which, name):
    """Bit for bit, whatever the magnitudes of the other images, also where one of those is not finite."""
    d, x, wt, b, dy = tensors(shape, 4300)
    assert route(d, which) == name
    base = product(d, which, x, wt, b, dy)
    for big in (np.float32(2.0 ** 60), np.float32(np.inf)):
        x2, dy2 = x.copy(), dy.copy()
        x2[1] *= big
        dy2[1] *= big
        with np.errstate(invalid="ignore"):
            got = product(d, which, x2, wt, b, dy2)
        others = np.arange(d.n) != 1
        assert np.array_equal(got[others], base[others])
        if np.isfinite(big) and which == DATA:
            assert np.array_equal(got[1], base[1] * big)
        assert np.isfinite(big) or not np.all(np.isfinite(got[1]))


def spread(a, axis, at, factor):
    """a, with its elements `at` along the axis multiplied."""
    out = a.copy()
    index = [slice(None)] * a.ndim
    index[axis] = at
    out[tuple(index)] *= np.float32(factor)
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("shape,which,name", ONE_EACH)
@pytest.mark.parametrize("case", ["contraction", "outputs", "one", "images"])
def test_magnitudes_the_terms_do_not_carry(shape, which, name, case):
    """Elements 2^-45 of the largest one under the same scale that carry the result, or a part of it: the pass then gives
    what the float kernel gives, every part of the result to the float tolerance of its own largest element."""
    d, x, wt, b, dy = tensors(shape, 4400)
    assert route(d, which) == name
    b = np.zeros_like(b)
    far, back = 2.0 ** 45, 2.0 ** -45
    parts = 1  # axis of the result whose entries are held each to its own magnitude
    if case == "contraction":  # a large channel (map) that meets small weights
        if which == FWD:
            x, wt = spread(x, 1, 0, far), spread(wt, 1, 0, back)
        elif which == DATA:
            dy, wt = spread(dy, 1, 0, far), spread(wt, 0, 0, back)
        else:  # a large image whose gradient is small
            x, dy = spread(x, 0, 0, far), spread(dy, 0, 0, back)
    elif case == "outputs":    # maps (channels) of the result far apart
        if which == FWD:
            wt = spread(wt, 0, 0, far)
        elif which == DATA:
            wt = spread(wt, 1, 0, far)
        else:
            dy, parts = spread(dy, 1, 0, far), 0
    elif case == "one":        # one large element, which meets zeros
        if which == FWD:
            x[:, 0, 0, 0] = far
            wt[:, 0] = 0
        elif which == DATA:
            dy[:, 0, 0, 0] = far
            wt[0] = 0
        else:
            x[0, 0, 0, 0] = far
            dy[0] = 0
    elif which == FILTER:      # images far apart: in both operands
        x, dy = spread(x, 0, 0, back), spread(dy, 0, 1, back)
    else:
        x, dy, parts = spread(x, 0, 0, far), spread(dy, 0, 0, far), 0
    got, want = product(d, which, x, wt, b, dy), expected(d, which, x, wt, b, dy)
    got, want = np.moveaxis(got, parts, 0), np.moveaxis(want, parts, 0)
    for i in range(got.shape[0]):
        assert_close(got[i], want[i], 2 * TOL, f"{case}: part {i}")


@pytest.mark.gpu
@pytest.mark.parametrize("shape,which,name", ONE_EACH)
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_non_finite_elements_stay_in_their_sums(shape, which, name, value):
    """One element of either operand is not finite: the sums it is part of are not, all others are what they were."""
    d, x, wt, b, dy = tensors(shape, 4500)
    assert route(d, which) == name
    base = product(d, which, x, wt, b, dy)
    first, second = {FWD: ("x", "w"), FILTER: ("x", "dy"), DATA: ("dy", "w")}[which]
    for operand in (first, second):
        t = {"x": x, "w": wt, "dy": dy}[operand]
        # the last row of the last image / map: where runs of rows and tiles end
        for at in ((t.shape[0] - 1, 1, t.shape[2] - 1, 0), (0, t.shape[1] - 1, 0, t.shape[3] - 1)):
            mark = {"x": np.ones_like(x), "w": np.ones_like(wt), "dy": np.ones_like(dy)}
            mark[operand] = np.zeros_like(t)
            mark[operand][at] = 1
            touched = expected(d, which, mark["x"], mark["w"], np.zeros_like(b), mark["dy"]) != 0
            spoilt = {"x": x, "w": wt, "dy": dy}
            spoilt[operand] = t.copy()
            spoilt[operand][at] = value
            got = product(d, which, spoilt["x"], spoilt["w"], b, spoilt["dy"])
            # (a sum of zeros counts: the unrolled product also multiplies the rectified zeros of x)
            assert not np.any(np.isfinite(got[touched]) & (got[touched] != 0) & (base[touched] != 0))
            if operand == second:  # the border's zeros as well: nothing is said of its map's other sums
                axis = 0 if which == FILTER else 1
                others = tuple(q for q in range(4) if q != axis)
                touched = np.broadcast_to(touched.any(axis=others, keepdims=True), touched.shape)
            rest = ~touched
            assert np.all(np.isfinite(got[rest]))
            assert np.max(np.abs(got - base)[rest], initial=0) <= 2 * TOL * np.max(np.abs(base))


@pytest.mark.gpu
@pytest.mark.parametrize("act", [vcnn.ACT_RELU, vcnn.ACT_TANH, vcnn.ACT_SIGMOID])
@pytest.mark.parametrize("shape,which,name", [t for t in ONE_EACH if t[1] == DATA])
def test_activation_derivative_of_declined_images(shape, which, name, act):
    """The derivative of the activation below is applied once, to the images the float kernel computes as to the others."""
    d, x, wt, b, dy = tensors(shape, 4550)
    assert route(d, which) == name
    dy[1, 0, 0, 0] = 2.0 ** 45
    wt[0] = 0
    y = np.tanh(x) * np.float32(0.7)
    ref = {vcnn.ACT_RELU: y > 0, vcnn.ACT_TANH: 1 - y.astype(np.float64) ** 2,
           vcnn.ACT_SIGMOID: y * (1 - y.astype(np.float64))}[act]
    want = expected(d, which, x, wt, b, dy) * ref
    yd, wd, dyd = (torch.from_numpy(a).to(DEV) for a in (y, wt, dy))
    ws = torch.full((vcnn.conv_workspace_bytes(d, which),), 255, dtype=torch.uint8, device=DEV)
    dx = torch.full(x.shape, float("nan"), device=DEV)
    vcnn.conv_bwd_data_act(d, act, yd, wd, dyd, dx, ws)
    dx = to_np(dx)
    for i in range(d.n):
        assert_close(dx[i], want[i], TOL, f"image {i}")


@pytest.mark.gpu
@pytest.mark.parametrize("shape,which,name", ONE_EACH)
def test_recorded_call_decides_anew_on_every_replay(shape, which, name):
    """A recorded pass on ordinary, far apart, non-finite and again ordinary data, with eager work between the replays."""
    d, x, wt, b, dy = tensors(shape, 4570)
    assert route(d, which) == name
    xd, wd, bd, dyd = (torch.from_numpy(a).to(DEV) for a in (x, wt, b, dy))
    ws = torch.empty(vcnn.conv_workspace_bytes(d, which), dtype=torch.uint8, device=DEV)
    out = torch.empty({FWD: dy, FILTER: wt, DATA: x}[which].shape, device=DEV)
    call = {FWD: lambda: vcnn.conv_fwd(d, xd, wd, bd, out, ws), DATA: lambda: vcnn.conv_bwd_data(d, wd, dyd, out, ws),
            FILTER: lambda: vcnn.conv_bwd_filter(d, xd, dyd, out, None, ws)}[which]
    call()
    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call()
    moved = {FWD: xd, FILTER: xd, DATA: dyd}[which]
    first = moved.clone()
    for value in (None, 2.0 ** 45, None, np.inf, np.nan, None):
        moved.copy_(first)
        if value is not None:
            moved[-1, -1, -1, -1] = value
        ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        assert np.isfinite(torch.randn(1 << 16, device=DEV).sum().item())  # unrelated eager work between replays
        call()
        torch.cuda.synchronize()
        assert torch.equal(torch.nan_to_num(got, 7.0, 8.0, 9.0), torch.nan_to_num(out, 7.0, 8.0, 9.0))


@pytest.mark.gpu
@pytest.mark.parametrize("shape,which,name", ONE_EACH)
def test_a_workspace_of_the_float_route_still_runs(shape, which, name):
    d, x, wt, b, dy = tensors(shape, 4600)
    small = float_bytes(d, which)
    assert route(d, which) == name and small < vcnn.conv_workspace_bytes(d, which)
    assert not vcnn.conv_route(d, which, small).startswith("two_term")
    got, want = (product(d, which, x, wt, b, dy, nbytes) for nbytes in (small, None))
    assert_close(got, want, 2 * TOL)


@pytest.mark.gpu
def test_batch_in_parts():
    """A layer whose re-laid copies exceed what a pass asks for goes through its batch in parts (a ragged last one), where
    the call brings a workspace for them; by its own query the forward pass and the input gradient run in float."""
    shape = (67, 64, 64, 64, 32, 5, 5, 2, 2)
    n, c, h, w, k, r, s, ph, pw = shape
    d, x, wt, b, dy = tensors(shape, 4700)
    need = [vcnn.conv_workspace_bytes(d, p) for p in range(3)]
    assert need[FWD] == 0 and need[FILTER] <= vcnn.conv_bwd_filter_noalloc_limit()
    assert [route(d, p) for p in range(2)] == ["implicit", IMPLICIT]
    sizes = ([256 << 20] * 3, [20 << 20, need[FILTER], 40 << 20])
    assert all(vcnn.conv_route(d, p, z[p]) == IMPLICIT for z in sizes for p in range(3))
    x[40, 0, 0, 0], dy[66, 0, 0, 0] = 2.0 ** 45, 2.0 ** 45  # declined: in a part of its own, in the ragged last one
    wt[:, 0, :, :], wt[0] = 0, 0
    whole, parts = ([run_pass(d, p, x, wt, b, dy, z[p]) for p in range(3)] for z in sizes)
    for p in (FWD, DATA):
        for img in range(n):
            assert_close(parts[p][img], whole[p][img], 2 * TOL)
    for img in (0, 40, 66):
        assert_close(parts[FWD][img:img + 1], O.conv_fwd(x[img:img + 1], wt, b, pad=(ph, pw)), TOL, "y")
        assert_close(parts[DATA][img:img + 1], O.conv_bwd_data(wt, dy[img:img + 1], (h, w), pad=(ph, pw)), TOL, "dx")
    # the kernel gradient's route depends on the shape alone: the same bits whatever more a caller has
    assert all(np.array_equal(p, q) for p, q in zip(parts[FILTER], whole[FILTER]))
    x[40, 0, 0, 0], dy[66, 0, 0, 0] = 1, 1  # (the same with nothing declined, against the float kernel)
    got = run_pass(d, FILTER, x, wt, b, dy)
    want = run_pass(d, FILTER, x, wt, b, dy, float_bytes(d, FILTER))
    assert_close(got[0], want[0], 2 * TOL, "dw")
    assert_close(got[1], want[1], 2 * TOL, "db")


@pytest.mark.gpu
def test_fold_in_parts():
    """The transposed product in two parts, the second one image shorter; declined images in both."""
    shape = (331, 357, 6, 11, 161, 6, 3, 0, 0)
    d, x, wt, b, dy = tensors(shape, 4800)
    assert route(d, DATA) == FOLD
    dy[3, 0, 0, 0] = dy[330, 0, 0, 0] = 2.0 ** 45
    wt[0] = 0
    got = product(d, DATA, x, wt, b, dy)
    for img in (0, 3, 165, 166, 329, 330):
        assert_close(got[img:img + 1], O.conv_bwd_data(wt, dy[img:img + 1], (d.h, d.w)), TOL, f"image {img}")


def test_the_query_asks_for_no_more_than_its_allowance():
    """No GPU needed: the workspace query of layers whose re-laid copies are large."""
    for shape in ((64, 64, 64, 64, 32, 5, 5, 2, 2), (512, 64, 64, 64, 64, 3, 3, 1, 1), (16, 38, 64, 64, 512, 16, 16, 0, 0)):
        assert vcnn.conv_workspace_bytes(vcnn.conv_desc(*shape), FWD) <= 64 << 20
    d = vcnn.conv_desc(*ONE_EACH[2][0])
    assert 0 < vcnn.conv_workspace_bytes(d, FILTER) <= vcnn.conv_bwd_filter_noalloc_limit()


def test_queries_and_routes_agree():
    """No GPU needed: over drawn layers every pass runs with exactly what its query asks for and with more, the kernel
    gradient by the same route; and the allocation-free entry point takes each layer whose float route fits it."""
    rng, seen = np.random.default_rng(5), set()
    log = lambda lo, hi: int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))
    for _ in range(400):
        r, s = (1, 1) if rng.random() < 0.2 else (log(1, 20), log(1, 20))
        d = vcnn.conv_desc(log(1, 400), log(5, 512), log(r, 100), log(s, 100), log(5, 512), r, s)
        for which in (FWD, FILTER, DATA):
            need = vcnn.conv_workspace_bytes(d, which)
            name = vcnn.conv_route(d, which, need)
            seen.add((which, name))
            for more in (need + 256, need + (64 << 20)):
                other = vcnn.conv_route(d, which, more)
                assert which != FILTER or other == name
            if name.startswith("two_term") and which == FILTER:
                limit = vcnn.conv_bwd_filter_noalloc_limit()
                assert (need <= limit) == (float_bytes(d, which) <= limit)
    assert {(FWD, IMPLICIT), (FILTER, IMPLICIT), (DATA, IMPLICIT), (DATA, FOLD), (FWD, "implicit")} <= seen


# bfloat16 layers whose input gradient is the transposed product on fragments (AUTO takes it where a correlation would
# leave the chip idle): ragged maps (padded steps), a kernel matrix and planes that end inside a tile, either order of adds
FOLD_BF16_SHAPES = [(6, 83, 14, 10, 286, 9, 9, 0, 0), (9, 60, 8, 8, 192, 5, 5, 2, 2), (7, 29, 143, 11, 142, 12, 10, 0, 0)]


@pytest.mark.parametrize("shape", FOLD_BF16_SHAPES)
def test_routes_of_the_bf16_layers(shape):
    assert route(vcnn.conv_desc(*shape, dtype=vcnn.BF16), DATA) == "fold_bf16"


@pytest.mark.gpu
@pytest.mark.parametrize("shape", FOLD_BF16_SHAPES)
def test_bf16_input_gradient_on_fragments(shape):
    n, c, h, w, k, r, s, ph, pw = shape
    d = vcnn.conv_desc(n, c, h, w, k, r, s, ph, pw, dtype=vcnn.BF16)
    oh, ow = vcnn.conv_out_shape(d)
    wt = bf16_round(random_tensor(4901, (k, c, r, s), scale=(2.0 / (k * r * s)) ** 0.5))
    dy, x = bf16_round(random_tensor(4902, (n, k, oh, ow))), bf16_round(random_tensor(4903, (n, c, h, w)))
    wd, dyd, xd = (torch.from_numpy(a).to(DEV).bfloat16() for a in (wt, dy, x))
    want = O.conv_bwd_data(wt, dy, (h, w), pad=(ph, pw))
    assert route(d, DATA) == "fold_bf16"
    ws = torch.full((vcnn.conv_workspace_bytes(d, DATA),), 255, dtype=torch.uint8, device=DEV)
    dx = torch.full((n, c, h, w), float("nan"), dtype=torch.bfloat16, device=DEV)
    vcnn.conv_bwd_data(d, wd, dyd, dx, ws)
    assert_close(to_np(dx.float()), want, 4e-3, "dx")  # one rounding of the result to eight bits
    vcnn.conv_bwd_data_act(d, vcnn.ACT_RELU, xd, wd, dyd, dx, ws)
    assert_close(to_np(dx.float()), np.where(x > 0, want, 0), 4e-3, "dx, ReLU below")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,name,shape", [(vcnn.F32, IMPLICIT, (9, 120, 62, 23, 5, 10, 3)),
                                              (vcnn.BF16, "implicit_bf16", (16, 512, 57, 10, 20, 5, 5))])
def test_kernel_gradient_with_a_run_shorter_than_the_waves_shares(dtype, name, shape):
    """A last run of output rows too short for every wave to get a slab, followed by the next image group in the same
    block: the waves without a share must not carry that run's fragments into the next one."""
    n, c, h, w, k, r, s = shape
    d = vcnn.conv_desc(n, c, h, w, k, r, s, dtype=dtype)
    assert route(d, FILTER) == name
    x = bf16_round(random_tensor(4801, (n, c, h, w)))
    dy = bf16_round(random_tensor(4802, (n, k, h - r + 1, w - s + 1)))
    t = torch.bfloat16 if dtype == vcnn.BF16 else torch.float32
    xd, dyd = (torch.from_numpy(a).to(DEV).to(t) for a in (x, dy))
    dw, db = torch.full((k, c, r, s), float("nan"), device=DEV), torch.full((k,), float("nan"), device=DEV)
    ws = torch.empty(vcnn.conv_workspace_bytes(d, vcnn.PASS_BWD_FILTER), dtype=torch.uint8, device=DEV)
    vcnn.conv_bwd_filter(d, xd, dyd, dw, db, ws)
    rdw, rdb = O.conv_bwd_filter(x, dy, (r, s))
    assert_close(to_np(dw), rdw, TOL, "dw")
    assert_close(to_np(db), rdb, TOL, "db")
