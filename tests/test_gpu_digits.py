"""The layer products on the integer matrix cores against 64-bit sums: ends of tiles, chunks and steps, what has to be summed again in double,
counts on the device, instances, rows that start anywhere."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# reduction, columns and rows (the smallest counts that the rule takes are somewhat lower): every kernel there is, columns for four to eight wavefronts
# and more than one block, last chunks of 1 to 64 k, rows that are no whole step
SHAPES = [(64, 256, 131_069), (62, 507, 131_072), (128, 128, 100_003), (100, 256, 65_533), (101, 505, 65_533), (192, 250, 30_577), (131, 512, 40_011),
          (256, 256, 28_399), (255, 101, 60_005), (256, 120, 90_001), (300, 127, 60_001), (257, 256, 60_001), (320, 510, 30_200), (512, 512, 8_191),
          (385, 126, 54_001), (450, 118, 90_000)]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch.device("cuda:0")


def product(what, A, W, out, **kw):
    from paper_2101_07706_amd import csgs
    (csgs.csgs_layer_gemm if what == "H" else csgs.csgs_layer_gemm_grad_z)(A, W, out, **kw)
    torch.cuda.synchronize()


def check(got, A, B):
    """One rounding to float (2^-24), whichever form sums; beside it 2^-52 of the summands each for the sums in double, here and there, and the least float."""
    A, B = A.double(), B.double()
    want = A @ B
    bound = 2.0 ** -24 * want.abs() + A.shape[1] * 2.0 ** -52 * (A.abs() @ B.abs()) + 2.0 ** -150
    d = (got.double() - want).abs()
    assert bool((d <= bound).all()), float((d / bound).nan_to_num().max())
    return float(d.norm()) / float(want.norm())


def operands(dev, what, K, N, M, seed, pad=0):
    g = torch.Generator(device=dev).manual_seed(seed)

    def matrix(r, c, x):
        t = torch.full((r, c + pad), float("nan"), device=dev)[:, :c] if pad else torch.empty((r, c), device=dev)
        t.copy_(x)
        return t
    A = torch.randn((M, K), generator=g, device=dev).clamp_min_(-0.5) * torch.randn((M, 1), generator=g, device=dev).exp_()
    W = torch.randn((K, N) if what == "H" else (N, K), generator=g, device=dev)
    return matrix(M, K, A), matrix(*W.shape, W), torch.full((M + 1, N + 3), float("nan"), device=dev)


@pytest.mark.parametrize("what", ["H", "dZ"])
@pytest.mark.parametrize("K,N,M", SHAPES)
def test_digit_products(dev, what, K, N, M):
    print(f"[digits] {what} {M} x {K} x {N}", flush=True)
    A, W, out = operands(dev, what, K, N, M, M + K + N, pad=M % 4)
    product(what, A, W, out[:M, :N])
    # a float's rounding is off by 2^-24 / sqrt(3) = 2^-24.8 of its unit, and the unit by 2^-0.4 of the value on average
    assert check(out[:M, :N], A, W if what == "H" else W.t().contiguous()) < 2.0 ** -25
    assert bool(torch.isnan(out[M:]).all()) and bool(torch.isnan(out[:, N:]).all()), "wrote outside"


# Row counts on the device: none, few (summed in double), half of a step, all
@pytest.mark.parametrize("what", ["H", "dZ"])
@pytest.mark.parametrize("m", [0, 1, 777, 5_000, 40_009, 65_536, 70_000])
def test_digit_products_device_count(dev, what, m):
    K, N, M = 256, 100, 65_536
    print(f"[digits] {what} {m} of {M}", flush=True)
    A, W, out = operands(dev, what, K, N, M, m)
    n = min(m, M)
    A[n:] = float("nan")
    product(what, A, W, out[:M, :N], M_dev=torch.tensor([m], dtype=torch.int32, device=dev))
    if n:
        check(out[:n, :N], A[:n], W if what == "H" else W.t().contiguous())
    assert bool(torch.isnan(out[n:]).all()) and bool(torch.isnan(out[:, N:]).all()), "wrote outside"


def test_digit_products_instances(dev):
    from paper_2101_07706_amd import csgs
    K, N, M, n_inst = 100, 256, 8_000, 8
    counts = [8_000, 0, 1, 7_999, 4_033, 8_000, 16, 6_000]
    print("[digits] instances", flush=True)
    A, W, _ = operands(dev, "H", K, N, M * n_inst, 3)
    A = A.reshape(n_inst, M, K)
    M_dev = torch.zeros((n_inst, 64), dtype=torch.int32, device=dev)
    M_dev[:, 0] = torch.tensor(counts, dtype=torch.int32)
    out = torch.full((n_inst, M, N), float("nan"), device=dev)
    nb = lambda t: t.stride(0) * t.element_size()
    csgs.csgs_layer_gemm(A[0], W, out[0], M_dev=M_dev[0, :1], inst=csgs.InstStrides(n_inst, 0, nb(M_dev), nb(A), 0, nb(out)))
    torch.cuda.synchronize()
    for k, n in enumerate(counts):
        if n:
            check(out[k, :n], A[k, :n], W)
        assert bool(torch.isnan(out[k, n:]).all()), "wrote outside"


# What the digits do not hold: outputs that all but cancel (in some rows, and in all, where whole tiles are summed again and blocks go on in double), rows and
# columns of zeros, of numbers beyond the exponents that are used, of one large number among small ones
@pytest.mark.parametrize("what", ["H", "dZ"])
@pytest.mark.parametrize("kind", ["cancel", "cancel_all", "zeros", "tiny", "huge", "spread"])
def test_digit_products_hard(dev, what, kind):
    K, N, M = 256, 256, 32_000
    print(f"[digits] {what} {kind}", flush=True)
    A, W, out = operands(dev, what, K, N, M, 5)
    B = W if what == "H" else W.t()
    if kind == "cancel":            # two halves that cancel but for their last bits, in one row in seven
        A[::7, 1::2] = -A[::7, ::2]
        B[1::2] = B[::2] * (1 + 2.0 ** -18)
    elif kind == "cancel_all":
        A[:, 1::2] = -A[:, ::2]
        B[1::2] = B[::2] * (1 + 2.0 ** -18)
    elif kind == "zeros":
        A[5::9], B[:, 3::5] = 0, 0
    elif kind == "tiny":
        A[::3] *= 2.0 ** -100
        B[:, 7] *= 2.0 ** -95
    elif kind == "huge":
        A[::3] *= 2.0 ** 90
        A[1] *= 2.0 ** 105
        B[:, 9] *= 2.0 ** 10
    else:                           # one feature a million times the others, with weights as much smaller
        A[:, 17] *= 2.0 ** 20
        B[17] *= 2.0 ** -20
        A[::2, 17] = 0
    product(what, A, W, out[:M, :N])
    check(out[:M, :N], A, B.contiguous())
    if kind == "zeros":
        assert bool((out[5:M:9, :N] == 0).all()) and bool((out[:M, 3:N:5] == 0).all())


# So many outputs that are small against row and column that blocks go on in double, where the last step lacks whole tiles of rows: one feature 300 times the
# others that no weight looks at, one output in fifty
@pytest.mark.parametrize("what", ["H", "dZ"])
@pytest.mark.parametrize("counted", [False, True])
@pytest.mark.parametrize("K,M", [(256, 65_537), (128, 100_003), (64, 131_069)])
def test_digit_products_many_listed(dev, what, counted, K, M):
    N = 256
    print(f"[digits] {what} {M} x {K} x {N} many small, counted {counted}", flush=True)
    A, W, out = operands(dev, what, K, N, M, 7)
    B = W if what == "H" else W.t()
    A[:, 5] *= 300
    B[5] = 0
    m = M - 40 if counted else M
    kw = dict(M_dev=torch.tensor([m], dtype=torch.int32, device=dev)) if counted else {}
    product(what, A, W, out[:M, :N], **kw)
    check(out[:m, :N], A[:m], B.contiguous())
    assert bool(torch.isnan(out[m:]).all()) and bool(torch.isnan(out[:, N:]).all()), "wrote outside"


@pytest.mark.parametrize("what", ["H", "dZ"])
def test_digit_products_infinite(dev, what):
    K, N, M = 256, 256, 32_000
    print(f"[digits] {what} infinite", flush=True)
    A, W, out = operands(dev, what, K, N, M, 6)
    B = W if what == "H" else W.t()
    A[100, 3], A[101, 255], A[31_999, 0], A[7] = float("inf"), float("nan"), float("-inf"), 0
    B[5, 40] = float("inf")
    product(what, A, W, out[:M, :N])
    want = (A.double() @ B.double().contiguous()).float()
    got = out[:M, :N]
    assert bool((torch.isnan(got) == torch.isnan(want)).all())
    odd = ~torch.isfinite(want)
    assert bool((got[odd & ~torch.isnan(want)] == want[odd & ~torch.isnan(want)]).all())
    rows = torch.ones(M, dtype=torch.bool, device=dev)
    rows[[100, 101, 31_999]] = False
    cols = torch.ones(N, dtype=torch.bool, device=dev)
    cols[40] = False
    check(got[rows][:, cols], A[rows], B[:, cols].contiguous())


def in_double(what, A, W, N):
    """The same rows in calls of few, which are summed in double whatever they hold."""
    out = torch.empty((A.shape[0], N), device=A.device)
    for i in range(0, A.shape[0], 512):
        product(what, A[i:i + 512], W, out[i:i + 512])
    return out


def same_bits(got, want):
    return bool(((got.contiguous().view(torch.int32) == want.view(torch.int32)) | (torch.isnan(got) & torch.isnan(want))).all())


# What a row gives depends on neither the other rows nor their number nor the form that these choose: both give the same bits
@pytest.mark.parametrize("what", ["H", "dZ"])
@pytest.mark.parametrize("K,N,M", SHAPES)
def test_digit_products_equal_double(dev, what, K, N, M):
    print(f"[digits] {what} {M} x {K} x {N} in both forms", flush=True)
    A, W, out = operands(dev, what, K, N, M, M + K, pad=M % 3)
    product(what, A, W, out[:M, :N])
    assert same_bits(out[:M, :N], in_double(what, A, W, N))


def hard(kind, A, B):
    """Operands that leave the digits little: A [M x K], B [K x N] are changed."""
    M, K = A.shape
    if kind == "repeated":            # equal values along k, whose roundings all point one way, and that all but cancel
        A.copy_(A[:, :1].expand(M, K).contiguous())
        B[::2] = B[:1].clone()
        B[1::2] = -B[:1] * (1 + 2.0 ** -18)
    elif kind == "one among many":    # the same in 2^-8 of the largest
        A.copy_(A[:, :1].expand(M, K).contiguous() * 2.0 ** -8)
        A[:, 3] *= 250
        B[::2] = B[:1].clone()
        B[1::2] = -B[:1] * (1 + 2.0 ** -10)
        B[3] = 0
    elif kind == "scales":            # features of very different size
        A *= torch.randn(K, generator=torch.Generator(device=A.device).manual_seed(1), device=A.device).mul_(4).exp_()
    elif kind == "weights of other scales":
        B *= torch.randn((K, 1), generator=torch.Generator(device=A.device).manual_seed(2), device=A.device).mul_(4).exp_()
    elif kind == "half way":          # sums that lie half way between two floats, or next to it
        A.copy_(torch.randint(-4096, 4096, A.shape, generator=torch.Generator(device=A.device).manual_seed(3), device=A.device).float())
        B.copy_(torch.randint(-4096, 4096, B.shape, generator=torch.Generator(device=A.device).manual_seed(4), device=A.device).float())
    elif kind == "sparse":
        A *= (torch.rand(A.shape, generator=torch.Generator(device=A.device).manual_seed(5), device=A.device) < 0.02)
        B *= (torch.rand(B.shape, generator=torch.Generator(device=A.device).manual_seed(6), device=A.device) < 0.1)
    elif kind == "least floats":      # results among the denormal numbers
        A *= 2.0 ** -75
        B *= 2.0 ** -70


@pytest.mark.parametrize("what", ["H", "dZ"])
@pytest.mark.parametrize("kind", ["repeated", "one among many", "scales", "weights of other scales", "half way", "sparse", "least floats"])
@pytest.mark.parametrize("K,N,M", [(64, 256, 131_069), (256, 256, 32_033), (512, 512, 8_191)])
def test_digit_products_equal_double_hard(dev, what, kind, K, N, M):
    print(f"[digits] {what} {M} x {K} x {N} {kind} in both forms", flush=True)
    A, W, out = operands(dev, what, K, N, M, K)
    hard(kind, A, W if what == "H" else W.t())
    product(what, A, W, out[:M, :N])
    assert same_bits(out[:M, :N], in_double(what, A, W, N))
    assert bool(torch.isnan(out[M:]).all()) and bool(torch.isnan(out[:, N:]).all()), "wrote outside"


# More to sum again than the list holds: worked off several times, then so much that the rest is done in double (from the first row on, from the middle on, in no step)
@pytest.mark.parametrize("what", ["H", "dZ"])
@pytest.mark.parametrize("dense_from", [0, 100_007, None])
@pytest.mark.parametrize("K,N,M", [(100, 256, 600_005), (260, 256, 200_009)])
def test_digit_products_list_worked_off(dev, what, dense_from, K, N, M):
    print(f"[digits] {what} {M} x {K} x {N} many listed, all from {dense_from}", flush=True)
    A, W, out = operands(dev, what, K, N, M, 11)
    B = W if what == "H" else W.t()
    A *= torch.randn(K, generator=torch.Generator(device=dev).manual_seed(7), device=dev).mul_(1.5).exp_()
    if dense_from is not None:
        A[dense_from:, 5] *= 3000
        B[5] = 0
    product(what, A, W, out[:M, :N])
    assert same_bits(out[:M, :N], in_double(what, A, W, N))
    assert bool(torch.isnan(out[M:]).all()) and bool(torch.isnan(out[:, N:]).all()), "wrote outside"


# Steps are counted over the rows that there are: instances of any number of rows one after the other, their outputs listed, rows beyond the counts of any value
@pytest.mark.parametrize("counts", [[16_000, 0, 33, 9_000, 16_000, 1, 0, 12_345], [0, 0, 0, 16_000], [27_000, 26_999, 0], [2_100] * 64])
@pytest.mark.parametrize("hard_values", [False, True])
@pytest.mark.parametrize("K", [100, 256])
def test_digit_products_steps_of_instances(dev, counts, hard_values, K):
    from paper_2101_07706_amd import csgs
    N, M, n_inst = 256, max(counts), len(counts)
    print(f"[digits] {n_inst} instances of {M} x {K} x {N}, hard {hard_values}", flush=True)
    A, W, _ = operands(dev, "H", K, N, M * n_inst, 13)
    A *= torch.randn(K, generator=torch.Generator(device=dev).manual_seed(8), device=dev).mul_(1.5).exp_()
    if hard_values:
        A[M // 2:, 5] *= 300
        W[5] = 0
    A = A.reshape(n_inst, M, K)
    M_dev = torch.zeros((n_inst, 64), dtype=torch.int32, device=dev)
    M_dev[:, 0] = torch.tensor(counts, dtype=torch.int32)
    for k, n in enumerate(counts):
        A[k, n:] = float("nan")
    out = torch.full((n_inst, M, N), float("nan"), device=dev)
    nb = lambda t: t.stride(0) * t.element_size()
    csgs.csgs_layer_gemm(A[0], W, out[0], M_dev=M_dev[0, :1], inst=csgs.InstStrides(n_inst, 0, nb(M_dev), nb(A), 0, nb(out)))
    torch.cuda.synchronize()
    for k, n in enumerate(counts):
        if n:
            assert same_bits(out[k, :n], in_double("H", A[k, :n], W, N)), k
        assert bool(torch.isnan(out[k, n:]).all()), "wrote outside"
