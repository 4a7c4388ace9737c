"""bf16 products at the edges of the 128x128 and 128x64 tiles and of their 32-deep K slices
(short last slices in both operand layouts, split K with a short last range),
against float64.

Element by element |C - ref| <= K 2^-24 (|A| |B|) for a float32 result (the
operands are exact in bf16, the sums float32), plus half a bf16 step of the
value where the result is bf16."""
import pytest

pytestmark = pytest.mark.gpu

# M, N, K: one past tiles; K of one short slice, of a multiple plus 8, 16 and 24; products whose
# cost model picks 128, 256x128 and 256x256 tiles with such K; last, two whose K-major form goes to
# the register-staged kernel, the second with K split
SHAPES = [(72, 72, 32), (136, 264, 40), (264, 136, 1000), (152, 768, 2312), (1032, 1048, 1048), (1768, 1024, 1784),
          (4104, 4096, 1064), (520, 6152, 4120),
          (136, 64, 1032), (1032, 40, 520), (1472, 3560, 1960), (1384, 400, 7032)]


@pytest.mark.parametrize("ak,bk", [(1, 0), (1, 1), (0, 0)])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_ragged(lib, M, N, K, ak, bk):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(M + 3 * N + 7 * K)
    A = torch.randn((M, K) if ak else (K, M), generator=g, device="cuda").bfloat16()
    B = torch.randn((N, K) if bk else (K, N), generator=g, device="cuda").bfloat16()
    # NaN right behind the operands: a short slice must not read on
    pad = lambda t: torch.cat([t.reshape(-1), torch.full((4096,), float("nan"), device="cuda", dtype=t.dtype)])
    Ap, Bp = pad(A), pad(B)
    f32 = 0 if ak else 1
    C = torch.full((M + 1, N), 7.0, device="cuda", dtype=torch.float32 if f32 else torch.bfloat16)
    n = lib.orbit_gemm_workspace_bytes(1, M, N, K, ak, bk)
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    lib.orbit_gemm(1, M, N, K, Ap, A.shape[1], ak, Bp, B.shape[1], bk, C, N, f32, 1.0, None, 0, ws)
    torch.cuda.synchronize()
    assert bool((C[M] == 7.0).all())
    a = (A if ak else A.t()).double()
    b = (B.t() if bk else B).double()
    ref = a @ b
    bound = K * 2.0 ** -24 * (a.abs() @ b.abs())
    if not f32:
        bound = bound * (1 + 2.0 ** -8) + ref.abs() * 2.0 ** -8
    assert bool(((C[:M].double() - ref).abs() <= bound).all())
