"""The bf16 convolution in chunks of channels: parity with the oracle at the edges of its tiles, chunks and rows."""
import pytest
import torch

from syno_inputs import BF16, F32, Builder, workloads as wl
from test_gpu_parity import run_all, syno  # noqa: F401  (fixture)

# tile configurations: 0 = waves along the pixels, 32 output channels; 1 = 64; 2 = 32, with 64 channels to a
# chunk, whose k-steps four waves share
CASES = {
    # 40 and 72 channels: a last chunk that is not full; blocks that cross images; an odd row that ends within an item of 4 pixels
    "ragged": (lambda: wl.make_conv(3, 40, 13, seed=71, bf16=True, Co=72, Wd=19, with_grad=True), ((0, 5), (0, 20), (1, 7), (2, 4), (2, 1)), (0, 1)),
    # a single chunk, rows as narrow as the kernel takes, blocks over many images
    "narrow": (lambda: wl.make_conv(9, 8, 5, seed=72, bf16=True, Co=16, Wd=4, with_grad=True), ((0, 1), (0, 45), (1, 31), (2, 12)), (0, 1)),
    # one to five chunks over the unrolled pairs; the most pixel tiles per wave, the last of them missing in some waves
    "three_chunks": (lambda: wl.make_conv(2, 96, 28, seed=73, bf16=True, Co=64, with_grad=True), ((0, 16), (0, 14), (1, 8), (2, 4)), (0, 1)),
    "four_chunks": (lambda: wl.make_conv(1, 128, 10, seed=74, bf16=True, Co=160, Wd=16, with_grad=True), ((0, 3), (1, 10), (2, 2)), (0, 1)),
    # two X items to a thread
    "wide": (lambda: wl.make_conv(1, 64, 9, seed=75, bf16=True, Co=40, Wd=60, with_grad=True), ((0, 8), (1, 4), (2, 1)), (0, 1)),
    # bf16 results; the runs of taps of backward-data begin at odd and at even elements
    "bf16_results": (lambda: wl.make_conv(2, 72, 9, seed=76, bf16=True, Co=56, Wd=11, with_grad=True, out_bf16=True), ((0, 9), (1, 4), (2, 3)), (0, 1)),
    # odd numbers of output channels, of results of backward-data, and the fewest of those that it takes
    "odd_channels_fwd": (lambda: wl.make_conv(2, 40, 7, seed=77, bf16=True, Co=37, Wd=9, with_grad=True), ((0, 3), (1, 14), (2, 2)), (0,)),
    "odd_channels_dx": (lambda: wl.make_conv(2, 37, 7, seed=78, bf16=True, Co=40, Wd=9, with_grad=True), ((0, 3), (1, 14), (2, 2)), (1,)),
    "three_channels_dx": (lambda: wl.make_conv(2, 3, 7, seed=83, bf16=True, Co=40, Wd=9, with_grad=True), ((0, 3), (1, 14), (2, 2)), (1,)),
    "two_channels_dx": (lambda: wl.make_conv(2, 2, 7, seed=84, bf16=True, Co=16, Wd=8, with_grad=True), ((0, 3), (1, 14), (2, 2)), (1,)),
    "stride2": (lambda: wl.make_conv(2, 64, 9, seed=79, bf16=True, Co=72, Wd=12, stride=2, with_grad=True), ((0, 5), (1, 4), (2, 3)), (0,)),
    "2x2": (lambda: wl.make_conv(3, 40, 13, seed=80, bf16=True, Co=72, Wd=19, K=2, with_grad=True), ((0, 5), (0, 20), (1, 7), (2, 4)), (1,)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name,cfg,rows", [(n, c, r) for n, v in CASES.items() for c, r in v[1]])
def test_parity_at_the_edges(syno, oracle, name, cfg, rows):  # noqa: F811
    make, _, directions = CASES[name]
    w = make()
    plan = syno.Plan(w.desc, mfma_variant=-2 - cfg, mfma_rows=rows)
    for which in directions:
        assert f"in-chunks tiles={cfg} rows/block={rows} " in plan.describe(which), plan.describe(which)
        assert plan.workspace_bytes(which) == 0
    run_all(syno, oracle, w, 0, directions=directions, mfma_variant=-2 - cfg, mfma_rows=rows)


def grouped_conv(N, groups, Cg, Og, H, W, out):
    """out[n,g,o,h,w] = sum X[n, g*Cg+c, h+kh-1, w+kw-1] * Wt[g,o,c,kh,kw], with the groups' output channels side by side."""
    b = Builder([("n", N), ("co", groups * Og), ("h", H), ("w", W)], name=f"grouped_conv3x3_g{groups}_{Cg}_to_{Og}_{H}x{W}_N{N}")
    g, o = b.merge(1, Og)
    gx, gw = b.share(g)
    (cx, cw), (khx, khw), (kwx, kww) = (b.share(b.reduce(n)) for n in (Cg, 3, 3))
    return b.finish([0, b.split(gx, cx), b.unfold(2, khx), b.unfold(3, kwx)], [gw, o, cw, khw, kww], BF16, out)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,rows", ((0, 5), (1, 4), (2, 2)))
@pytest.mark.parametrize("N,groups,Cg,Og,H,W,out,directions", [
    (3, 2, 40, 48, 9, 7, F32, (0, 1)),       # a last chunk and last panels that are not full; blocks over two images
    (4, 2, 64, 64, 14, 14, BF16, (0, 1)),    # a plane of tiles per group that is dealt to the XCDs (configurations 0 and 2)
    (2, 3, 24, 37, 7, 10, F32, (0,)),        # an odd number of results of a group
    (2, 3, 37, 24, 7, 10, BF16, (1,)),       # the same of backward-data: each group's last run of taps is read from one element before it
    (3, 4, 3, 16, 6, 8, F32, (1,)), (3, 5, 2, 8, 5, 9, F32, (1,)),
])
def test_groups(syno, oracle, N, groups, Cg, Og, H, W, out, directions, cfg, rows):  # noqa: F811
    d = grouped_conv(N, groups, Cg, Og, H, W, out)
    xs, ws, os_ = (N, groups * Cg, H, W), (groups, Og, Cg, 3, 3), (N, groups * Og, H, W)
    st = wl.Stream(85)
    w = wl._finish(d, xs, ws, os_, st.normal(xs), st.uniform_pm(1.0 / (9 * Cg) ** 0.5, ws), st.normal(os_), Cg * 9)
    plan = syno.Plan(d, mfma_variant=-2 - cfg, mfma_rows=rows)
    assert plan.x_shape == xs and plan.out_shape == os_
    for which in directions:
        assert f"in-chunks tiles={cfg} rows/block={rows} " in plan.describe(which), plan.describe(which)
    run_all(syno, oracle, w, 0, directions=directions, mfma_variant=-2 - cfg, mfma_rows=rows)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", (0, 1, 2))
def test_what_lies_beside_the_operands(syno, cfg):  # noqa: F811
    """Infinities and NaNs reach the results that they are a term of and no others (40 channels: the last chunk reads the
    last octet in the place of those that it does not have); what lies before and behind the operands does not."""
    d = wl.conv2d(2, 40, 40, 5, 6, 3, 3, BF16, F32)
    plan, plain = syno.Plan(d, mfma_variant=-2 - cfg, mfma_rows=2), syno.Plan(d, kernel_policy=1)
    assert "in-chunks" in plan.describe(0) and "in-chunks" in plan.describe(1)
    gen = torch.Generator(device="cuda").manual_seed(6)

    def at(shape, first):
        n = torch.Size(shape).numel()
        flat = torch.full((n + 2 * first,), float("nan"), dtype=torch.bfloat16, device="cuda")
        t = flat[first:first + n].view(shape)
        t.copy_(torch.randn(shape, generator=gen, device="cuda") / 8)
        return t

    X, W, G = (at(shape, 8) for shape in (plan.x_shape, plan.w_shape, plan.out_shape))
    X[0, 39, 2, 2], X[1, 32, 0, 0], G[0, 39, 4, 5], G[1, 35, 1, 1] = float("inf"), float("nan"), float("inf"), float("nan")
    for a, b in ((plan.forward(X, W), plain.forward(X, W)), (plan.backward_data(G, W), plain.backward_data(G, W))):
        assert torch.equal(torch.isfinite(a), torch.isfinite(b)) and torch.equal(torch.isnan(a), torch.isnan(b))
        fine = torch.isfinite(b)
        # 360 products, exact in fp32, in any order on either side: 2 * 360 roundings of sums below 360 * max|X| * max|W|
        assert float((a - b)[fine].abs().max()) <= 2 * 360 * 2.0 ** -24 * float(b[fine].abs().max()) * 8


@pytest.mark.gpu
@pytest.mark.parametrize("H,W", [(8, 12), (7, 9), (5, 16)])
@pytest.mark.parametrize("kind", ("f32", "bf16", "bf16_results"))
def test_input_gradients_of_strided_convolutions_are_stored_as_the_image(syno, oracle, H, W, kind):  # noqa: F811
    """3x3 with stride 2 on 2x2 windows of the phase planes: lanes side by side hold the two phases of a row and exchange halves where
    rows are whole quads (12 and 16 pixels), else store every second pixel."""
    w = wl.make_conv(32 if kind == "f32" else 3, 96, H, seed=81, bf16=kind != "f32", Co=192, Wd=W, stride=2, with_grad=True, out_bf16=kind == "bf16_results")
    plan = syno.Plan(w.desc)
    assert " stores the phase planes of dX as the image, " in plan.describe(1), plan.describe(1)
    assert "(window=2): " in plan.describe(1) and ("bf16-parts" if kind == "f32" else "in-chunks") in plan.describe(1), plan.describe(1)
    run_all(syno, oracle, w, 0, directions=(1,))
    if kind == "f32":
        # infinities and NaNs are summed again, from results that the lane beside has stored
        plain = syno.Plan(w.desc, kernel_policy=1)
        gen = torch.Generator(device="cuda").manual_seed(9)
        G, V = torch.randn(plan.out_shape, generator=gen, device="cuda"), torch.randn(plan.w_shape, generator=gen, device="cuda") / 40
        G[0, 3, 2, 5], G[1, 7, H - 1, W - 1], G[31, 9, 0, 0] = float("inf"), float("nan"), float("-inf")
        a, b = plan.backward_data(G, V), plain.backward_data(G, V)
        # (the taps that a 2x2 window on the planes has and the 3x3 one has not are products with zero: NaN beside an infinity)
        fine = torch.isfinite(a)
        assert bool(torch.isfinite(b)[fine].all()) and int((~fine).sum()) <= 3 * 96 * 16
        # up to 4 * 192 terms in fp32 on either side
        assert float((a - b)[fine].abs().max()) <= 2 * 768 * 2.0 ** -24 * 8 * float(b[fine].abs().max())


@pytest.mark.gpu
@pytest.mark.parametrize("N,C,Co,H,W", [(60, 42, 8, 14, 26), (13, 160, 24, 11, 13), (32, 70, 64, 16, 22)])
def test_input_gradients_of_strided_convolutions_with_few_channels(syno, oracle, N, C, Co, H, W):  # noqa: F811
    """One chunk of 8 or 24 channels, and two; output channels that fill no panel; rows of whole and of broken quads."""
    w = wl.make_conv(N, C, H, seed=82, bf16=True, Co=Co, Wd=W, stride=2, with_grad=True)
    describe = syno.Plan(w.desc).describe(1)
    assert "(window=2): mfma_contraction_bf16 in-chunks " in describe, describe
    run_all(syno, oracle, w, 0, directions=(1,))


@pytest.mark.gpu
@pytest.mark.parametrize("H,N", [(7, 9001), (8, 8200)])
@pytest.mark.parametrize("kind,options", [("in-chunks", {"mfma_variant": -2}), ("bf16-parts", {"mfma_variant": -2}), ("variant=4", {"mfma_variant": 5})])
def test_more_than_65536_tiles(syno, H, N, kind, options):  # noqa: F811
    """A block finds its tile by multiplying with a reciprocal, which is one off for some numbers from 2^16 tiles on if it is not put right.
    Rows per block do not change a result's sums."""
    d = wl.conv2d(N, 8 if kind == "in-chunks" else 32, 80, H, 8, 3, 3, BF16 if kind == "in-chunks" else F32, F32)
    many, few = (syno.Plan(d, mfma_rows=rows, **options) for rows in (1, H))
    assert f"{kind} " in many.describe(0) and "rows/block=1 " in many.describe(0), many.describe(0)
    assert int(many.describe(0).split("grid=")[1].split()[0]) > 65536
    gen = torch.Generator(device="cuda").manual_seed(11)
    X, W = (torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16 if kind == "in-chunks" else torch.float32) for shape in (many.x_shape, many.w_shape))
    assert torch.equal(many.forward(X, W), few.forward(X, W))
