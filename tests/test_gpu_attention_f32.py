"""float32 attention on both sides of the rule that gives small grids 32-row
blocks (up to 64, 128 or 191 blocks of 128 rows by head_dim, direction and
length), against float64.

Lengths around the 32-row tiles and the four waves' turns of 128 rows; q, k, v,
dO and the gradients have different row strides and NaN in the columns past
the heads, so a kernel that reads or writes past a slice shows.

Bound: every result is a chain of float32 sums of at most dh + L terms, so its
error is below (dh + L + 16) 2^-24 times the same chain of magnitudes (16 for
the exponential and the scalings); a logit's error enters a probability as a
relative one."""
import pytest

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 1, 32), (1, 2, 31, 64), (2, 1, 33, 128), (1, 3, 127, 32), (1, 2, 129, 64), (2, 2, 300, 128),
         (1, 2, 1030, 64), (3, 63, 128, 32), (3, 64, 128, 32), (2, 96, 129, 64),
         (1, 64, 40, 128), (1, 65, 40, 128), (1, 129, 40, 128), (1, 128, 72, 64), (1, 129, 72, 64), (1, 192, 72, 32),
         (1, 63, 300, 64), (1, 64, 300, 32)]


@pytest.mark.parametrize("B,H,L,dh", CASES)
def test_attention_f32(lib, B, H, L, dh):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(B + 3 * H + 7 * L + dh)
    A, T = H * dh, B * L

    def padded(ld):
        x = torch.full((T, ld), float("nan"), device="cuda")
        x[:, :A] = torch.randn((T, A), generator=g, device="cuda")
        return x

    q, k, v, dO = padded(A + 8), padded(2 * A), padded(A + 24), padded(A + 16)
    o, o32 = torch.zeros(T, A, device="cuda"), torch.zeros(T, A + 8, device="cuda")
    lse = torch.zeros(B, H, L, device="cuda")
    grads = [torch.full((T, A + 32), float("nan"), device="cuda") for _ in range(3)]
    lib.orbit_attention_fwd(0, B, H, L, dh, q, q.shape[1], k, k.shape[1], v, v.shape[1], o, A, lse, o32, A + 8)
    ws = torch.zeros(lib.orbit_attention_bwd_workspace_bytes(B, H, L, dh), dtype=torch.uint8, device="cuda")
    lib.orbit_attention_bwd(0, B, H, L, dh, q, q.shape[1], k, k.shape[1], v, v.shape[1], o32, A + 8, 1, lse,
                            dO, dO.shape[1], *grads, A + 32, ws)
    torch.cuda.synchronize()
    hd = lambda x: x[:, :A].double().reshape(B, L, H, dh).transpose(1, 2).contiguous()
    Q, K, V, G = hd(q), hd(k), hd(v), hd(dO)
    S = (Q @ K.transpose(2, 3).contiguous()) * dh ** -0.5
    P = S.softmax(-1)
    ref = P @ V
    dP = G @ V.transpose(2, 3).contiguous()
    dS = P * (dP - (G * ref).sum(-1, keepdim=True)) * dh ** -0.5
    tr = lambda x: x.transpose(2, 3).contiguous()
    # magnitudes: of the logits (+ 1: relative errors of P), of dP - D, of dS
    mS = 1 + (Q.abs() @ tr(K.abs())) * dh ** -0.5
    mP = P * mS
    mG = (G.abs() @ tr(V.abs())) + (G.abs() * (mP @ V.abs())).sum(-1, keepdim=True)
    mdS = mP * mG * dh ** -0.5

    def check(name, got, want, mag):
        ratio = float(((got - want).abs() / mag).max()) / ((dh + L + 16) * 2.0 ** -24)
        assert ratio <= 1, f"{name}: {ratio:.2f} of the bound"

    check("o", hd(o), ref, mP @ V.abs())
    assert torch.equal(o, o32[:, :A])
    check("lse", lse.double(), S.logsumexp(-1), mS.max(-1).values)
    for name, got, want, mag in zip(("dq", "dk", "dv"), grads, (dS @ K, tr(dS) @ Q, tr(P) @ G),
                                    (mdS @ K.abs(), tr(mdS) @ Q.abs(), tr(mP) @ G.abs())):
        check(name, hd(got), want, mag)
        assert bool(got[:, A:].isnan().all()), name


def test_attention_f32_infinite_logits(lib):
    """Keys whose logits are -inf for a query weigh nothing, also when they
    fill the first tiles of the sweep."""
    import torch
    L, dh = 300, 32
    q = torch.ones(L, dh, device="cuda") * 1e30
    k = torch.ones(L, dh, device="cuda")
    k[:160] = -1e30
    k[160:] = 1e-30
    v = torch.arange(L, device="cuda").float()[:, None].expand(L, dh).contiguous()
    o, lse = torch.zeros(L, dh, device="cuda"), torch.zeros(1, 1, L, device="cuda")
    lib.orbit_attention_fwd(0, 1, 1, L, dh, q, dh, k, dh, v, dh, o, dh, lse, None, 0)
    torch.cuda.synchronize()
    want = float(v[160:, 0].mean())
    assert float((o - want).abs().max()) <= 140 * 2.0 ** -24 * L
