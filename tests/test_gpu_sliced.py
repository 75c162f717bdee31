"""fp32 matrix products in slices of their reduction, against fp64, and with values that bf16 parts cannot stand for."""
import pytest
import torch

from syno_inputs import workloads as wl
from test_gpu_parity import syno  # noqa: F401  (fixture)

# M, N, K and the calls that are sliced: an odd number of rows; each call; a last chunk that starts early; one chunk or two a
# slice; a result that is no multiple of four; most slices
SHAPES = ((333, 896, 448, (1,)), (1312, 1600, 1344, (0, 1, 2)), (264, 1032, 200, (1, 2)), (1040, 256, 128, (2,)), (4104, 37, 129, (2,)),
          (72, 2560, 576, (1,)), (8192, 256, 256, (2,)))


def sliced(plan):
    return tuple(which for which in range(3) if "slices of the reduction" in plan.describe(which))


@pytest.mark.parametrize("M,N,K,calls", SHAPES)
def test_which_calls_are_sliced(M, N, K, calls):
    import paper_2410_23745_amd as s
    p = s.Plan(wl.matmul(M, N, K))
    assert sliced(p) == calls, [p.describe(which) for which in range(3)]
    assert p.workspace_bytes(2) <= 32 << 20          # (the scratch of the entry point without a workspace)
    assert sliced(s.Plan(wl.matmul(M, N, K), mfma_splits=2)) == ()


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,calls", SHAPES)
def test_against_fp64(syno, M, N, K, calls):  # noqa: F811
    """A result is off by a rounding for each term of a k-step of 32, step and slice, and by the products that the parts leave
    out (less than a rounding of their term)."""
    p = syno.Plan(wl.matmul(M, N, K))
    gen = torch.Generator(device="cuda").manual_seed(9)
    X, W, G = (torch.randn(*shape, generator=gen, device="cuda") for shape in ((M, K), (K, N), (M, N)))
    for which in calls:
        a, b = ((X, W), (G, W.t()), (X.t(), G))[which]
        got = p.forward(X, W) if which == 0 else p.backward_data(G, W) if which == 1 else p.backward_weight(X, G)
        a, b = a.double().contiguous(), b.double().contiguous()
        bound = (a.abs() @ b.abs()) * ((34 + a.shape[1] / 32 + 32) * 2.0 ** -24)
        assert bool(((got.double() - a @ b).abs() <= bound).all()), which


@pytest.mark.gpu
def test_infinities_and_nans(syno):  # noqa: F811
    """One infinity and one NaN in different slices: where the fp64 product has them."""
    M, N, K, calls = SHAPES[1]
    p = syno.Plan(wl.matmul(M, N, K))
    gen = torch.Generator(device="cuda").manual_seed(10)
    X, W, G = (torch.randn(*shape, generator=gen, device="cuda") for shape in ((M, K), (K, N), (M, N)))
    X[3, 5], X[M - 2, K - 1], G[7, 2], G[M - 1, N - 1] = float("inf"), float("nan"), float("-inf"), float("nan")
    for got, want in ((p.forward(X, W), X.double() @ W.double()), (p.backward_data(G, W), G.double() @ W.double().t().contiguous()),
                      (p.backward_weight(X, G), X.double().t().contiguous() @ G.double())):
        assert torch.equal(torch.isnan(got), torch.isnan(want))
        assert torch.equal(torch.isposinf(got), torch.isposinf(want)) and torch.equal(torch.isneginf(got), torch.isneginf(want))
