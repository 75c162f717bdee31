"""The fp32 contraction on the bf16 matrix cores (every value split into three bf16 parts): parity with the oracle at the
edges of its tiles, chunks and stages, and the values that parts cannot stand for."""
import numpy as np
import pytest
import torch

from syno_inputs import F32, workloads as wl
from test_gpu_parity import run_all, syno  # noqa: F401  (fixture)
from util import assert_close, to_dev, to_host, tol_for

# tile configurations: 0 = 64 output channels, 1 = 32 with the taps of a window dealt to two waves, 2 = to four,
# 3 = 128 output channels of a 1x1 window
CASES = {
    # 40 channels: a last chunk that starts early; blocks that cross images; 72 output channels: a block of 8
    "3x3_ragged": (lambda: wl.make_conv(3, 40, 13, seed=31, Co=72, Wd=19, with_grad=True), ((0, 5), (1, 7), (2, 4), (2, 1)), (0, 1)),
    # one chunk, an image narrower than a quad of pixels, one pixel tile for four rows of waves
    "3x3_narrow": (lambda: wl.make_conv(5, 32, 6, seed=32, Co=36, Wd=2, with_grad=True), ((0, 1), (0, 30), (1, 11), (2, 12)), (0, 1)),
    # the most pixel tiles per wave, the last of them missing in some waves
    "3x3_full_tiles": (lambda: wl.make_conv(2, 96, 28, seed=33, Co=64, with_grad=True), ((0, 14), (1, 14), (2, 4)), (0, 1)),
    # channel counts that are only even
    "3x3_even_channels": (lambda: wl.make_conv(2, 34, 9, seed=34, Co=38, Wd=11, with_grad=True), ((1, 9), (2, 4)), (0, 1)),
    "3x3_stride2": (lambda: wl.make_conv(2, 64, 9, seed=35, Co=72, Wd=12, stride=2, with_grad=True), ((0, 5), (1, 4), (2, 3)), (0,)),
    "1x1": (lambda: wl.make_conv(3, 72, 10, seed=36, Co=136, Wd=15, K=1, with_grad=True), ((3, 1), (3, 13)), (0, 1)),
    # cyclic rows whose shift depends on the group, 1x3 window
    "cyclic_1x3": (lambda: wl.make_gshift(3, seeds=(37, 37, 37), with_grad=True, C=144, H=9, Wd=11, bf16=False), ((0, 4), (1, 9)), (0, 1)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name,cfg,rows", [(n, c, r) for n, v in CASES.items() for c, r in v[1]])
def test_parity_at_the_edges(syno, oracle, name, cfg, rows):  # noqa: F811
    make, _, directions = CASES[name]
    w = make()
    plan = syno.Plan(w.desc, mfma_variant=-2 - cfg, mfma_rows=rows)
    for which in directions:
        assert f"bf16-parts tiles={cfg} rows/block={rows} " in plan.describe(which), plan.describe(which)
        assert plan.workspace_bytes(which) == 0
    run_all(syno, oracle, w, 0, directions=directions, mfma_variant=-2 - cfg, mfma_rows=rows)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", (0, 1, 2))
def test_values_that_parts_do_not_stand_for(syno, cfg):  # noqa: F811
    """Infinities, NaNs, values near the largest float, subnormal operands and results: as the index-program kernel has them."""
    d = wl.conv2d(2, 40, 48, 10, 12)
    parts, plain = syno.Plan(d, mfma_variant=-2 - cfg), syno.Plan(d, kernel_policy=1)
    assert "bf16-parts" in parts.describe(0) and "bf16-parts" in parts.describe(1)
    gen = torch.Generator(device="cuda").manual_seed(5)
    X, W = torch.randn(parts.x_shape, generator=gen, device="cuda"), torch.randn(parts.w_shape, generator=gen, device="cuda") / 20

    def agree(x, w):
        for a, b in ((parts.forward(x, w), plain.forward(x, w)),):
            assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isposinf(a), torch.isposinf(b))
            assert torch.equal(torch.isneginf(a), torch.isneginf(b))
            fine = torch.isfinite(b)
            # 360 terms in fp32 on either side; the largest subnormal step for results that are subnormal themselves
            err, bound = (a - b)[fine].double().abs(), 2e-5 * b[fine].double().abs().max() + 2e-45 * 400
            assert float(err.max()) <= float(bound)

    Y, V = X.clone(), W.clone()
    Y[0, 3, 5, 5], Y[0, 39, 0, 0], Y[1, 7, 9, 11], Y[1, 8, 4, 4], Y[1, 9, 4, 4] = float("inf"), float("-inf"), float("nan"), float("inf"), float("-inf")
    agree(Y, W)
    V[3, 4, 1, 1], V[40, 0, 0, 2] = float("inf"), float("nan")
    agree(X, V)
    Z = X.clone()
    Z[0, 0, 2, 2] = 3.4e38            # rounds to infinity as a bf16 value
    agree(Z, W * 1e-3)
    for scale in (1e30, 1e-30, 1e-36, 1e-41):
        agree(X * scale, W)
    agree(torch.zeros_like(X), W)


# backward-weight: widths that divide by 8 (rows without a zero between them), 4, 2 and nothing; one chunk per workgroup and
# many; images smaller than a chunk; channel counts inside a block; the windows it has; a bound on the workgroups
DW_CASES = {
    "3x3_w8": (lambda: wl.make_conv(3, 40, 11, seed=41, Co=72, Wd=8, with_grad=True), (0, 1, 5)),
    "3x3_w56": (lambda: wl.make_conv(2, 32, 7, seed=42, Co=70, Wd=56, with_grad=True), (0, 3)),
    "3x3_w20": (lambda: wl.make_conv(3, 33, 6, seed=43, Co=64, Wd=20, with_grad=True), (0, 2)),
    "3x3_w14": (lambda: wl.make_conv(4, 35, 5, seed=44, Co=65, Wd=14, with_grad=True), (0, 7)),
    "3x3_w7": (lambda: wl.make_conv(9, 64, 7, seed=45, Co=130, Wd=7, with_grad=True), (0, 4)),
    "3x3_one_row": (lambda: wl.make_conv(31, 16, 1, seed=46, Co=24, Wd=5, with_grad=True), (0, 1)),
    "3x3_wide": (lambda: wl.make_conv(1, 24, 3, seed=47, Co=40, Wd=199, with_grad=True), (0, 2)),
    "1x1_w10": (lambda: wl.make_conv(3, 72, 10, seed=48, Co=136, Wd=10, K=1, with_grad=True), (0, 3)),
    "1x1_w16": (lambda: wl.make_conv(5, 65, 3, seed=49, Co=63, Wd=16, K=1, with_grad=True), (0, 1)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name,groups", [(n, g) for n, v in DW_CASES.items() for g in v[1]])
def test_weight_gradient_parity_at_the_edges(syno, oracle, name, groups):  # noqa: F811
    w = DW_CASES[name][0]()
    assert "bf16-parts" in syno.Plan(w.desc, dw_workgroups=groups).describe(2)
    run_all(syno, oracle, w, 0, directions=(2,), dw_workgroups=groups)


def weight_sums(x, g, KH, KW):
    """The weight gradient of a convolution with zero padding, tap by tap."""
    (C, H, W), O = x.shape[1:], g.shape[1]
    x = torch.nn.functional.pad(x, (KW // 2, KW // 2, KH // 2, KH // 2))
    return torch.stack([torch.stack([g.transpose(0, 1).reshape(O, -1) @ x[:, :, a:a + H, b:b + W].transpose(0, 1).reshape(C, -1).t().contiguous()
                                     for b in range(KW)], -1) for a in range(KH)], -2)


@pytest.mark.gpu
@pytest.mark.parametrize("KH,KW", ((3, 1), (1, 3)))
@pytest.mark.parametrize("N,C,O,H,W", ((2, 64, 64, 9, 30), (3, 72, 80, 12, 21), (4, 65, 63, 1, 24), (5, 100, 40, 5, 6)))
def test_weight_gradient_of_one_sided_windows(syno, N, C, O, H, W, KH, KW):  # noqa: F811
    """Against the sum of its terms in fp64.  Every term is within 2^-22 of its product's size (nine parts less the three
    smallest), a chunk's sum of 64 is rounded twice, and the chunks and splits (fewer than 64 here) add up in fp32."""
    p = syno.Plan(wl.conv2d(N, C, O, H, W, KH, KW))
    assert "bf16-parts" in p.describe(2)
    gen = torch.Generator(device="cuda").manual_seed(6)
    X, G = torch.randn(p.x_shape, generator=gen, device="cuda"), torch.randn(p.out_shape, generator=gen, device="cuda")
    got = p.backward_weight(X, G).double()

    whole, size = weight_sums(X.double(), G.double(), KH, KW), weight_sums(X.double().abs(), G.double().abs(), KH, KW)
    assert bool(((got - whole).abs() <= size * (2.0 ** -22 + 64 * 2.0 ** -24)).all())


@pytest.mark.gpu
@pytest.mark.parametrize("groups", (0, 1))
def test_weight_gradient_of_values_that_parts_do_not_stand_for(syno, groups):  # noqa: F811
    d = wl.conv2d(2, 40, 48, 10, 12)
    parts, plain = syno.Plan(d, dw_workgroups=groups), syno.Plan(d, kernel_policy=1)
    assert "bf16-parts" in parts.describe(2)
    gen = torch.Generator(device="cuda").manual_seed(7)
    X, G = torch.randn(parts.x_shape, generator=gen, device="cuda"), torch.randn(parts.out_shape, generator=gen, device="cuda") / 20

    def agree(x, g):
        a, b = parts.backward_weight(x, g), plain.backward_weight(x, g)
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isposinf(a), torch.isposinf(b))
        assert torch.equal(torch.isneginf(a), torch.isneginf(b))
        fine = torch.isfinite(b)
        # 240 terms in fp32 on either side; the largest subnormal step for results that are subnormal themselves
        assert float((a - b)[fine].double().abs().max()) <= 2e-5 * float(b[fine].double().abs().max()) + 2e-45 * 300

    Y, V = X.clone(), G.clone()
    Y[0, 3, 5, 5], Y[0, 39, 0, 0], Y[1, 7, 9, 11] = float("inf"), float("-inf"), float("nan")
    agree(Y, G)
    V[0, 3, 1, 1], V[1, 40, 0, 2] = float("inf"), float("nan")
    agree(X, V)
    Z = X.clone()
    Z[0, 0, 2, 2] = 3.4e38            # rounds to infinity as a bf16 value
    agree(Z, G * 1e-3)
    for scale in (1e30, 1e-30, 1e-36, 1e-41):
        agree(X * scale, G)
    agree(torch.zeros_like(X), G)


def test_where_the_planner_takes_it():
    import paper_2410_23745_amd as s
    for C, H in wl.RESNET18_STAGES:
        p = s.Plan(wl.conv2d(32, C, C, H, H))
        assert all("bf16-parts" in p.describe(which) for which in (0, 1, 2))
    # rows that would be mostly filling, one chunk of pixels, a window it does not have
    for d in (wl.conv2d(32, 64, 64, 56, 4), wl.conv2d(1, 1024, 1024, 7, 7), wl.conv2d(32, 64, 64, 56, 56, 1, 5)):
        assert "bf16-parts" not in s.Plan(d).describe(2)
    # too little work for it, a window or weight layout that it does not have, a named variant of the other kernel
    for p in (s.Plan(wl.conv2d(1, 16, 16, 16, 16)), s.Plan(wl.conv2d(32, 64, 64, 56, 56, 5, 5)),
              s.Plan(wl.conv2d(32, 64, 64, 28, 28, 3, 3, F32, F32, (1, 0, 2, 3))), s.Plan(wl.conv2d(32, 64, 64, 28, 28), mfma_variant=4, mfma_rows=7)):
        assert all("bf16-parts" not in p.describe(which) for which in (0, 1))


def test_weights_out_of_reach_of_a_lane_offset():
    """A workgroup's weights are addressed by 32-bit byte offsets from its first one: output channels (or, in the adjoint,
    forward output channels) so far apart that the last of a tile lies 4 GiB on are not its work."""
    import paper_2410_23745_amd as s
    # 24 channels of a chunk apart: 24 * stride * 4 bytes reach 2^32 at 44739243 weights per channel
    for d, which in ((wl.matmul(40, 16, 48234496), 2), (wl.conv2d(1, 50331648, 40, 5, 5, 1, 1), 1)):
        assert "bf16-parts" not in s.Plan(d).describe(which)
    for d in (wl.matmul(40, 16, 44739232), wl.conv2d(1, 44739232, 40, 5, 5, 1, 1)):
        assert any("bf16-parts" in s.Plan(d).describe(which) for which in (1, 2))
    # 127 output channels of a tile apart: 127 * stride + 24 weights reach 2^30 at 8454661 weights each
    far, near = wl.conv2d(1, 8454664, 128, 3, 3, 1, 1), wl.conv2d(1, 8454656, 128, 3, 3, 1, 1)
    assert "bf16-parts" not in s.Plan(far, mfma_variant=-5).describe(0) and "bf16-parts" in s.Plan(near, mfma_variant=-5).describe(0)
    # (channels that the tile has no more of do not count)
    assert "bf16-parts" in s.Plan(wl.conv2d(1, 8454664, 40, 3, 3, 1, 1), mfma_variant=-5).describe(0)


def least_time(call, n=5):
    """us between events, the least of n calls"""
    best = float("inf")
    for _ in range(n + 1):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.gpu
@pytest.mark.parametrize("scale", (1e-25, 1e-30, 1e-37, 1e-40))
def test_small_values_are_ordinary_ones(syno, scale):  # noqa: F811
    """Values down to the subnormal ones have whole parts: every result is within 2^-22 of the size of its terms (nine parts
    less the three smallest, sums of 32 or 64 terms rounded twice, at most 64 of them here), and of 2^-149 times the partial
    sums that are stored as subnormals; and no call takes another way for them, which would be a hundred times slower."""
    p = syno.Plan(wl.conv2d(8, 64, 64, 28, 28), mfma_variant=-2)
    assert all("bf16-parts" in p.describe(which) for which in range(3))
    gen = torch.Generator(device="cuda").manual_seed(9)
    X, G, W = (torch.randn(s, generator=gen, device="cuda") for s in (p.x_shape, p.out_shape, p.w_shape))
    x, g = X * scale, G * scale
    calls = (lambda x, g: p.forward(x, W), lambda x, g: p.backward_data(g, W), lambda x, g: p.backward_weight(X, g))
    conv = torch.nn.functional.conv2d

    def weight_sums(a, b):
        return conv(a.transpose(0, 1).contiguous(), b.transpose(0, 1).contiguous(), padding=1).transpose(0, 1)

    Wb = W.flip(2, 3).transpose(0, 1).contiguous()
    for which, (a, b, sums) in enumerate(((x, W, lambda a, b: conv(a, b, padding=1)), (g, Wb, lambda a, b: conv(a, b, padding=1)), (X, g, weight_sums))):
        a, b = a.double().cpu(), b.double().cpu()
        got, whole, size = calls[which](x, g).double().cpu(), sums(a, b), sums(a.abs(), b.abs())
        assert bool(((got - whole).abs() <= size * (2.0 ** -22 + 64 * 2.0 ** -24) + 300 * 2.0 ** -149).all()), which
        slow, plain = least_time(lambda: calls[which](x, g)), least_time(lambda: calls[which](X, G))
        assert slow <= 4 * plain + 50, (which, slow, plain)


def same_as_the_definition(got, plain, size, terms):
    """got: a result; plain: the index program's, which sums a result's terms in order in fp32; size: its sums of the terms'
    magnitudes.  Infinities and NaNs are the same, other values within the roundings of both sums."""
    assert torch.equal(torch.isnan(got), torch.isnan(plain)) and torch.equal(torch.isposinf(got), torch.isposinf(plain))
    assert torch.equal(torch.isneginf(got), torch.isneginf(plain))
    fine = torch.isfinite(plain) & torch.isfinite(size)
    assert bool(((got - plain).double().abs() <= size.double() * (2 * terms * 2.0 ** -24) + terms * 2.0 ** -149)[fine].all())


def odd_values(a, b):
    """Pairs like (a, b) with values that parts do not stand for, in either operand and in both."""
    gen = torch.Generator().manual_seed(11)

    def at(t, *values):
        t = t.clone()
        t.view(-1)[torch.randperm(t.numel(), generator=gen)[:len(values)].to(t.device)] = torch.tensor(values, device=t.device)
        return t
    inf, nan = float("inf"), float("nan")
    yield at(a, inf), b
    yield at(a, inf, -inf, nan, 3.4e38, -3e38), b * 1e-3
    yield a, at(b, inf)
    yield a, at(b, -inf, nan, 3e38)
    yield a * 1e-3, at(b, *([nan, inf] * 20))
    yield at(a, inf, 3e38), at(b, 1e-40, 1e-39)
    yield a * 1e30, b
    yield a, b * 1e32
    yield a * float("nan"), b


# every tap's way through the sums of whole tiles: reversed taps, a stride, cyclic rows by group, one-sided windows, 1x1
ODD_CASES = {
    "3x3": (lambda: wl.conv2d(2, 40, 48, 10, 12), (0, 1, 2), (0, 1)),
    "3x3_one_column": (lambda: wl.conv2d(5, 32, 36, 6, 1), (0, 2), (0, 1)),
    "3x3_stride2": (lambda: wl.conv2d(2, 40, 48, 6, 7, stride=2), (0, 1, 2), (0,)),
    "3x1": (lambda: wl.conv2d(3, 36, 52, 7, 9, 3, 1), (0, 1), (0, 1)),
    "1x1": (lambda: wl.conv2d(3, 72, 136, 7, 9, 1, 1), (3,), (0, 1)),
    "cyclic_1x3": (lambda: wl.grouped_shift_unfold(3, 144, 144, 9, 11, 4, 3, F32, F32), (0, 1), (0, 1)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name,cfg", [(n, c) for n, v in ODD_CASES.items() for c in v[1]])
def test_tiles_with_results_that_parts_cannot_give(syno, name, cfg):  # noqa: F811
    make, _, directions = ODD_CASES[name]
    parts, plain = syno.Plan(make(), mfma_variant=-2 - cfg), syno.Plan(make(), kernel_policy=1)
    gen = torch.Generator(device="cuda").manual_seed(12)
    W = torch.randn(parts.w_shape, generator=gen, device="cuda") / 20
    for which in directions:
        assert f"bf16-parts tiles={cfg} " in parts.describe(which)
        A = torch.randn(parts.x_shape if which == 0 else parts.out_shape, generator=gen, device="cuda")
        for a, w in odd_values(A, W):
            got, ref, size = ((p.forward if which == 0 else p.backward_data)(x, y) for p, x, y in ((parts, a, w), (plain, a, w), (plain, a.abs(), w.abs())))
            same_as_the_definition(got, ref, size, parts.free_size(which))


@pytest.mark.gpu
@pytest.mark.parametrize("W", (7, 8, 12, 14))
@pytest.mark.parametrize("KH,KW", ((3, 3), (3, 1), (1, 3), (1, 1)))
@pytest.mark.parametrize("groups", (0, 1, 3))
def test_weight_gradient_tiles_with_results_that_parts_cannot_give(syno, W, KH, KW, groups):  # noqa: F811
    d = wl.conv2d(3, 40, 72, 9, W, KH, KW)
    parts, plain = syno.Plan(d, dw_workgroups=groups), syno.Plan(d, kernel_policy=1)
    assert "bf16-parts" in parts.describe(2)
    gen = torch.Generator(device="cuda").manual_seed(13)
    X, G = torch.randn(parts.x_shape, generator=gen, device="cuda"), torch.randn(parts.out_shape, generator=gen, device="cuda") / 20
    for x, g in odd_values(X, G):
        same_as_the_definition(parts.backward_weight(x, g), plain.backward_weight(x, g), plain.backward_weight(x.abs(), g.abs()), parts.free_size(2))


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ("one infinity", "beyond the parts", "all NaN"))
def test_values_that_parts_do_not_stand_for_are_no_cliff(syno, kind):  # noqa: F811
    """A tile is summed again by the fp32 matrix instructions, not by its lanes one result at a time (a hundred times the
    ordinary call's time and more)."""
    p = syno.Plan(wl.conv2d(16, 64, 64, 56, 56))
    assert all("bf16-parts" in p.describe(which) for which in range(3))
    gen = torch.Generator(device="cuda").manual_seed(14)
    X, G, W = (torch.randn(s, generator=gen, device="cuda") for s in (p.x_shape, p.out_shape, p.w_shape))

    def odd(t):
        if kind == "beyond the parts":
            return t * 1e30
        t = t.clone()
        if kind == "all NaN":
            return t.fill_(float("nan"))
        t.view(-1)[t.numel() // 3] = float("inf")
        return t
    x, g = odd(X), odd(G)
    for which, (slow, plain) in enumerate(((lambda: p.forward(x, W), lambda: p.forward(X, W)), (lambda: p.backward_data(g, W), lambda: p.backward_data(G, W)),
                                           (lambda: p.backward_weight(X, g), lambda: p.backward_weight(X, G)))):
        t, t0 = least_time(slow), least_time(plain)
        print(f"[time] {kind} pass {which}: {t0:.0f} -> {t:.0f} us", flush=True)
        assert t <= 10 * t0 + 50, (kind, which, t, t0)


# strided, rows wider than the fp32 instructions' kernel stages: the phase planes of X and the spread weights need 40 MB
WIDE_STRIDED = dict(N=28, C=21, H=38, seed=51, Co=11, Wd=59, stride=2, with_grad=True)


def test_which_calls_without_a_workspace_keep_the_index_program():
    import paper_2410_23745_amd as s
    f = WIDE_STRIDED
    p = s.Plan(wl.conv2d(f["N"], f["C"], f["Co"], f["H"], f["Wd"], stride=2))
    assert p.kernel(2) == "mfma_contraction_phases" and p.workspace_bytes(2) > 32 << 20
    assert p.describe(2).endswith("(without a workspace: index program)")
    # the scratch is enough; the fp32 instructions have the stride-1 problem too (never taken without a workspace)
    for d in (wl.conv2d(2, 21, 11, 38, 59, stride=2), wl.conv2d(64, 64, 128, 56, 56, stride=2)):
        assert s.Plan(d).kernel(2) == "mfma_contraction_phases" and "without a workspace" not in s.Plan(d).describe(2)


@pytest.mark.gpu
def test_weight_gradient_without_a_workspace_beyond_the_scratch(syno, oracle):  # noqa: F811
    """The entry point without a workspace takes the call on the index program, whatever the other one does."""
    w = wl.make_conv(**WIDE_STRIDED)
    p = syno.Plan(w.desc)
    X, G = to_dev(w.X, w.X_bits), to_dev(w.G, w.G_bits)
    got = {"workspace": p.backward_weight(X, G), "static": torch.full(p.w_shape, float("nan"), device="cuda")}
    p.backward_weight_static(X, G, got["static"])
    _, dw = oracle.backward(w.desc, w.X, w.W, w.G, False, True)
    _, mdw = oracle.backward(w.desc, np.abs(w.X), np.abs(w.W), np.abs(w.G), False, True)
    for name, v in got.items():
        assert_close(to_host(v), dw, mdw, p.free_size(2), False, "backward-weight " + name, tol_for(w.desc))


# (N, C, O, H, W): whole rows of 7 and of 14 pixels, pixels by four, by two and single; several chunks per workgroup
FP32_DW_CASES = ((33, 40, 72, 7, 7), (9, 64, 65, 14, 14), (2, 32, 70, 30, 28), (4, 24, 40, 21, 10), (3, 33, 64, 23, 13))


@pytest.mark.gpu
@pytest.mark.parametrize("KH,KW", ((3, 3), (3, 1), (1, 3), (1, 1)))
@pytest.mark.parametrize("groups", (1, 3))
@pytest.mark.parametrize("N,C,O,H,W", FP32_DW_CASES)
def test_weight_gradient_on_the_fp32_instructions(syno, N, C, O, H, W, KH, KW, groups):  # noqa: F811
    """A named variant of the fp32 contraction kernel keeps the weight gradient on the fp32 instructions, which tensors of 2 GiB
    and more have it on.  A sum rounds once per term and workgroup."""
    p = syno.Plan(wl.conv2d(N, C, O, H, W, KH, KW), mfma_variant=1, mfma_rows=1, dw_workgroups=groups)
    chunks, splits = (int(p.describe(2).split(k + "=")[1].split()[0]) for k in ("chunks", "splits"))
    assert "bf16-parts" not in p.describe(2) and chunks > splits, p.describe(2)
    gen = torch.Generator(device="cuda").manual_seed(16)
    X, G = torch.randn(p.x_shape, generator=gen, device="cuda"), torch.randn(p.out_shape, generator=gen, device="cuda")
    got = p.backward_weight(X, G).double()
    whole, size = weight_sums(X.double(), G.double(), KH, KW), weight_sums(X.double().abs(), G.double().abs(), KH, KW)
    assert bool(((got - whole).abs() <= size * ((N * H * W + 3) * 2.0 ** -24)).all())


def test_named_choices_of_the_fp32_kernels():
    import paper_2410_23745_amd as s
    d = wl.conv2d(32, 64, 64, 28, 28)
    assert all("bf16-parts" in s.Plan(d).describe(which) for which in range(3))
    taps = s.Plan(d, mfma_taps=1)
    assert all("taps/row-step=1 " in taps.describe(which) for which in (0, 1)), (taps.describe(0), taps.describe(1))
    named = s.Plan(d, mfma_variant=4, mfma_rows=7)
    assert "variant=3 " in named.describe(0) and "bf16-parts" not in named.describe(2)
    assert "bf16-parts tiles=1 " in s.Plan(d, mfma_variant=-3, mfma_taps=1).describe(0)
    # rows that the fp32 instructions' kernel does not stage
    wide = wl.conv2d(1, 24, 40, 3, 199)
    assert "bf16-parts" in s.Plan(wide, mfma_variant=1, mfma_rows=1).describe(2)
