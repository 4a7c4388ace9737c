"""float32 products on split bf16 matrix instructions and on 32x32 tiles: edges
of tiles and K slices in every layout against float64, and operands holding
infinities and NaN.

The bound is the float32 one: |C - ref| <= K 2^-24 (|A| |B|) element by element
(K sums rounded to 24 bits each; the kernels round fewer)."""
import pytest

pytestmark = pytest.mark.gpu

# M, N, K: below and above the 32x32-tile limits (M N K of 5.5e8, K of 1024, 2048 tiles, few rows
# of 1024 K-major floats); one past tiles
# and slices, a single slice, K not a multiple of 16, K split over blocks, 64-wide tiles
SHAPES = [(8, 8, 8), (40, 72, 24), (264, 136, 512), (520, 1032, 1024), (2056, 136, 2008), (1024, 1024, 1096),
          (136, 264, 16 * 1024), (4104, 64, 2056), (2016, 1024, 64), (2048, 1024, 64), (40, 4104, 1024), (24, 8200, 1024)]


def _operands(torch, M, N, K, ak, bk):
    g = torch.Generator(device="cuda")
    g.manual_seed(M * 7 + N * 3 + K)
    A = torch.randn((M, K) if ak else (K, M), generator=g, device="cuda")
    B = torch.randn((N, K) if bk else (K, N), generator=g, device="cuda")
    return A, B


def _run(lib, torch, A, B, M, N, K, ak, bk):
    C = torch.full((M + 1, N), 7.0, device="cuda")  # a guard row behind the result
    n = lib.orbit_gemm_workspace_bytes(0, M, N, K, ak, bk)
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    lib.orbit_gemm(0, M, N, K, A, A.shape[1], ak, B, B.shape[1], bk, C, N, 1, 1.0, None, 0, ws)
    torch.cuda.synchronize()
    assert bool((C[M] == 7.0).all())
    return C[:M]


@pytest.mark.parametrize("ak,bk", [(1, 0), (1, 1), (0, 0)])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_f32(lib, M, N, K, ak, bk):
    import torch
    A, B = _operands(torch, M, N, K, ak, bk)
    a = (A if ak else A.t()).double()
    b = (B.t() if bk else B).double()
    C = _run(lib, torch, A, B, M, N, K, ak, bk)
    worst = ((C.double() - a @ b).abs() / (a.abs() @ b.abs())).max().item()
    assert worst <= K * 2.0 ** -24, worst


# 32x32 tiles; 128x128 with K split, and unsplit; 64x64
FALLBACK = [(40, 48, 64), (1032, 1032, 1032), (2056, 2056, 1032), (4104, 64, 2056)]


@pytest.mark.parametrize("ak,bk", [(1, 0), (1, 1), (0, 0)])
@pytest.mark.parametrize("M,N,K", FALLBACK)
def test_gemm_f32_not_finite(lib, M, N, K, ak, bk):
    """Infinities and NaN reach exactly the outputs that float32 arithmetic gives
    them, with the same sign; everything else stays finite and right. Values at
    the top of the float32 range, which bf16 rounding would overflow, stay finite."""
    import torch
    A, B = _operands(torch, M, N, K, 1, 0)
    B = B.abs()
    A[3, 5], A[7, 9], A[9, 1], A[11, 2] = float("inf"), float("nan"), float("-inf"), 3.4e38
    B[2] = 1e-3
    a, b = A.double(), B.double()
    C = _run(lib, torch, A if ak else A.t().contiguous(), B.t().contiguous() if bk else B, M, N, K, ak, bk)
    ref = a @ b
    ok = torch.isfinite(ref)
    assert torch.equal(ok, torch.isfinite(C))
    assert torch.equal(torch.isnan(ref), torch.isnan(C))
    inf = torch.isinf(ref)
    assert torch.equal(torch.sign(ref[inf]), torch.sign(C[inf].double()))
    a[~torch.isfinite(a)] = 0
    err = ((C.double() - ref).abs() / (a.abs() @ b.abs()))[ok].max().item()
    assert err <= K * 2.0 ** -24, err


@pytest.mark.parametrize("ak,bk", [(1, 0), (1, 1), (0, 0)])
@pytest.mark.parametrize("M,N,K", FALLBACK)
@pytest.mark.parametrize("rows,sa,sb", [("one", -126, 0), ("all", -126, 0), ("one", 116, -20), ("all", 55, 50)])
def test_gemm_f32_range(lib, M, N, K, ak, bk, rows, sa, sb):
    """Operands near the bottom of the float32 range, whose parts unscaled would
    fall below the smallest bf16, and operands or products near its top, which
    overflow when scaled, keep their 24 bits: the results' errors stay those of
    K roundings that add up like a random walk."""
    import torch
    A, B = _operands(torch, M, N, K, 1, 0)
    i = 37 if rows == "one" else slice(None)
    A[i] *= 2.0 ** sa
    B *= 2.0 ** sb
    C = _run(lib, torch, A if ak else A.t().contiguous(), B.t().contiguous() if bk else B, M, N, K, ak, bk)
    ref = A.double() @ B.double()
    for r in (i, 38):
        err = ((C.double() - ref)[r].norm() / ref[r].norm()).item()
        assert err <= K ** 0.5 * 2.0 ** -24, err


@pytest.mark.parametrize("ak,bk", [(1, 0), (1, 1), (0, 0)])
@pytest.mark.parametrize("x", [1 + 511 / 65536, 1 + 2.0 ** -8 - 2.0 ** -17])
def test_gemm_f32_split_bound(lib, x, ak, bk):
    """Operands whose second and third parts are the largest there are, all of
    one sign, and a single 16-deep step: each product keeps all but 2^-24 of
    itself, and the two sums are rounded, once each, and added."""
    import torch
    M, N, K = 6016, 6016, 16
    A = torch.full((M, K) if ak else (K, M), x, device="cuda")
    B = torch.full((N, K) if bk else (K, N), x, device="cuda")
    C = _run(lib, torch, A, B, M, N, K, ak, bk)
    ref = K * x * x
    assert float((C.double() - ref).abs().max()) <= 3 * 2.0 ** -24 * ref


@pytest.mark.parametrize("ak", [0, 1])
@pytest.mark.parametrize("ld,tiny", [(1500000, True), (5500000, False)])
def test_gemm_f32_wide_rows(lib, ak, ld, tiny):
    """The 32x32 kernel's loads run past K by up to 206 rows, at 32-bit offsets:
    it is taken only where those cannot wrap back into the operand."""
    import torch
    M, N, K = 40, 72, 8
    buf = torch.empty((K - 1) * ld + 80, device="cuda")
    a, b = _operands(torch, M, N, K, 1, 0)
    if ak:
        A, lda = a, K
    else:
        A, lda = torch.empty((K - 1) * ld + M, device="cuda"), ld
        torch.as_strided(A, (K, M), (ld, 1)).copy_(a.t())
    torch.as_strided(buf, (K, N), (ld, 1)).copy_(b)
    C = torch.zeros(M, N, device="cuda")
    ws = torch.empty(max(16, lib.orbit_gemm_workspace_bytes(0, M, N, K, ak, 0)), dtype=torch.uint8, device="cuda")
    lib.orbit_timing_filter(None)
    lib.orbit_timing_enable(True)
    lib.orbit_gemm(0, M, N, K, A, lda, ak, buf, ld, 0, C, N, 1, 1.0, None, 0, ws)
    torch.cuda.synchronize()
    names = lib.orbit_timing_kernel_names()
    lib.orbit_timing_enable(False)
    assert ("gemm_f32_tiny" in names) == tiny, names
    ref = a.double() @ b.double()
    assert float(((C.double() - ref).abs() / (a.double().abs() @ b.double().abs())).max()) <= K * 2.0 ** -24
