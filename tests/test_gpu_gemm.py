"""bf16 matrix products on their operands as they lie: every layout at the edges of its tiles, steps and splits, against fp64."""
import pytest
import torch

from syno_inputs import BF16, F32, workloads as wl
from test_gpu_parity import syno  # noqa: F401  (fixture)

# M, N, K: less than a piece of a tile; one past a tile and a step; ragged in all three; several splits of the reduction
# (and more splits than the last has steps for); the largest tile, ragged; many tile rows
SHAPES = ((8, 128, 64), (129, 136, 72), (100, 64, 192), (257, 200, 328), (7, 3072, 2056), (3000, 128, 136), (2056, 2312, 776), (8200, 200, 128))


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("out", (F32, BF16))
def test_products_and_gradients(syno, M, N, K, out):  # noqa: F811
    """A result is a sum of exact products, rounded at most once per term of a step of 64 and once per step and split; a bf16
    result once more."""
    p = syno.Plan(wl.matmul(M, N, K, BF16, out))
    gen = torch.Generator(device="cuda").manual_seed(8)

    def operand(*shape):
        return torch.randn(*shape, generator=gen, device="cuda").bfloat16()
    X, W, G = operand(M, K), operand(K, N), operand(M, N)
    for which in range(2 if out == BF16 else 3):
        assert " as it is: " in p.describe(which)
        a, b, got = ((X, W, p.forward), (G, W.t(), p.backward_data), (X.t(), G, p.backward_weight))[which]
        got = (got(X, W) if which == 0 else got(G, W) if which == 1 else got(X, G)).double()
        a, b = a.double().contiguous(), b.double().contiguous()
        bound = (a.abs() @ b.abs()) * ((64 + a.shape[1] / 64 + 64) * 2.0 ** -24)
        whole = a @ b
        if out == BF16:
            bound = bound + whole.abs() * 2.0 ** -8
        assert bool(((got - whole).abs() <= bound).all()), (which, float(((got - whole).abs() - bound).max()))


def test_which_products_are_taken():
    import paper_2410_23745_amd as s
    seen = set()
    for M, N, K in SHAPES:
        d = [s.Plan(wl.matmul(M, N, K, BF16, F32)).describe(which) for which in range(3)]
        assert all(" as it is: " in x for x in d)
        seen |= {x.split("tiles=")[1].split()[0] + ("" if x.endswith("reduction-splits=1") else " split") for x in d}
    assert {x.split()[0] for x in seen} == {"256x192", "128x192", "128x128"} and any("split" in x for x in seen), seen
    # fp32 operands, an axis that is no multiple of 8, a named number of splits
    for p in (s.Plan(wl.matmul(256, 256, 256)), s.Plan(wl.matmul(256, 256, 252, BF16, F32)), s.Plan(wl.matmul(256, 256, 256, BF16, F32), mfma_splits=2)):
        assert all(" as it is: " not in p.describe(which) for which in range(3))


@pytest.mark.parametrize("M,N,K", ((11136, 8432, 200), (23992, 17816, 96), (16136, 13584, 216), (16384, 2048, 768), (10240, 1536, 2048)))
def test_sums_of_the_weight_gradients_splits_fit_the_static_scratch(M, N, K):
    """The entry point without a workspace has 32 MiB (it took the first three on the convolution kernels too)."""
    import paper_2410_23745_amd as s
    p = s.Plan(wl.matmul(M, N, K, BF16, F32))
    assert " as it is: " in p.describe(2) and p.workspace_bytes(2) <= 32 << 20
