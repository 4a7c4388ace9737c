"""The streaming aggregation kernels (bf16, 8 or 16 heads, embeddings up to
2048) against the fp64 oracle at the sizes where they can go wrong: embeddings
around each instantiation's width and not filling it, variables around the
16-row slots and at the ends of the range, fewer patches than blocks and
several patches per block; and just outside the range, where the general path
runs."""
import numpy as np
import pytest

import oracle as O
import synth
from helpers import TOL, check, dev, host

pytestmark = pytest.mark.gpu

CASES = [
    # B, L, V, d, heads, head_dim
    (1, 5, 16, 512, 16, 32),       # exactly one slot per patch
    (2, 300, 17, 256, 8, 32),      # patches > blocks, a one-row last slot, half-empty columns
    (1, 530, 3, 520, 8, 24),       # just past 512 columns; fewer variables than a slot
    (1, 40, 48, 1024, 16, 64),
    (1, 33, 49, 1032, 16, 16),     # just past 1024 columns
    (1, 20, 31, 1544, 8, 64),      # just past 1536 columns
    (1, 12, 128, 2048, 16, 32),    # the largest V and d
    (1, 270, 2, 2040, 16, 8),
    (3, 7, 97, 8, 8, 8),           # the smallest d; few columns: general path
    (1, 9, 16, 64, 8, 8),          # the fewest columns of the streaming kernels
    (1, 9, 15, 64, 16, 8),         # just fewer
    (1, 9, 129, 512, 8, 32),       # V past the range: general path
    (1, 9, 20, 2056, 16, 32),      # d past the range: general path
]


@pytest.mark.parametrize("case", CASES)
def test_agg_stream(lib, case):
    import torch
    from paper_2404_14712_amd._lib import AggDesc
    B, L, V, d, H, dh = case
    c = synth.small_config("115m", dtype="bf16", B=B, L=L, V=V, d=d, agg_heads=H, agg_head_dim=dh, sigma=0.1)
    tok = synth.normal(c.seed, "tok", (B, L, V, d), dtype="bf16")
    prm = synth.make_params(c.seed, "agg", synth.agg_param_shapes(d, H * dh, L), 0.1, "bf16")
    dz = synth.normal(c.seed, "dz", (B, L, d), dtype="bf16")
    desc = AggDesc(B, L, V, d, H, dh, 1)
    pd = {k: dev(v, "bf16") for k, v in prm.items()}
    tokd, dzd = dev(tok, "bf16"), dev(dz, "bf16")
    z = torch.zeros(B, L, d, dtype=torch.bfloat16, device="cuda")
    # scratch with NaN bit patterns: nothing unwritten may be read
    saved = torch.full((lib.orbit_var_aggregate_saved_bytes(desc),), 255, dtype=torch.uint8, device="cuda")
    ws = torch.full((lib.orbit_var_aggregate_workspace_bytes(desc),), 255, dtype=torch.uint8, device="cuda")
    # a guard row behind the gradient: no store may pass the last patch
    dtok = torch.full((B * L * V + 1, d), 7.0, dtype=torch.bfloat16, device="cuda")
    g = {k: torch.full(v.shape, 7.0, dtype=torch.float32, device="cuda") for k, v in prm.items()}
    lib.orbit_var_aggregate(desc, tokd, pd, z, saved, ws)
    lib.orbit_var_aggregate_bwd(desc, tokd, pd, saved, dzd, dtok, g, 0, ws)
    torch.cuda.synchronize()
    ref, cache = O.agg_fwd(tok, prm, H)
    rdtok, rg = O.agg_bwd(dz, cache, prm)
    tol = TOL["bf16"]
    check("z", host(z), ref, tol)
    check("dtok", host(dtok[:-1]).reshape(rdtok.shape), rdtok, tol)
    assert bool((dtok[-1] == 7.0).all())
    for k in rg:
        check(f"d{k}", host(g[k]), rg[k], tol, floor_ref=rg["b_q"])


def _token_gradient(lib, tok, prm, dz, H, dh):
    """dtok of the library, of the oracle, and the oracle's weights."""
    import torch
    from paper_2404_14712_amd._lib import AggDesc
    B, L, V, d = tok.shape
    desc = AggDesc(B, L, V, d, H, dh, 1)
    pd = {k: dev(v, "bf16") for k, v in prm.items()}
    tokd, dzd = dev(tok, "bf16"), dev(dz, "bf16")
    z = torch.zeros(B, L, d, dtype=torch.bfloat16, device="cuda")
    saved = torch.full((lib.orbit_var_aggregate_saved_bytes(desc),), 255, dtype=torch.uint8, device="cuda")
    ws = torch.full((lib.orbit_var_aggregate_workspace_bytes(desc),), 255, dtype=torch.uint8, device="cuda")
    dtok = torch.zeros(B * L * V, d, dtype=torch.bfloat16, device="cuda")
    g = {k: torch.zeros(v.shape, dtype=torch.float32, device="cuda") for k, v in prm.items()}
    lib.orbit_var_aggregate(desc, tokd, pd, z, saved, ws)
    lib.orbit_var_aggregate_bwd(desc, tokd, pd, saved, dzd, dtok, g, 0, ws)
    torch.cuda.synchronize()
    _, cache = O.agg_fwd(tok, prm, H)
    rdtok, _ = O.agg_bwd(dz, cache, prm)
    return host(dtok).reshape(rdtok.shape), rdtok, cache["a"]


def _case(B, L, V, d, H, dh, sigma):
    c = synth.small_config("115m", dtype="bf16", B=B, L=L, V=V, d=d, agg_heads=H, agg_head_dim=dh, sigma=sigma)
    tok = synth.normal(c.seed, "tok", (B, L, V, d), dtype="bf16")
    prm = synth.make_params(c.seed, "agg", synth.agg_param_shapes(d, H * dh, L), sigma, "bf16")
    dz = synth.normal(c.seed, "dz", (B, L, d), dtype="bf16")
    return c, tok, prm, dz


@pytest.mark.parametrize("V", [17, 40])
def test_agg_stream_large_value_bias(lib, V):
    """A value bias far above the value outputs: the token gradient does not see
    it (the weights sum to one), so the bound is the usual one."""
    H, dh = 8, 64
    _, tok, prm, dz = _case(1, 24, V, 512, H, dh, 0.1)
    prm["b_v"] = np.full_like(prm["b_v"], 4096.0) * np.sign(prm["b_v"])
    got, ref, _ = _token_gradient(lib, tok, prm, dz, H, dh)
    check("dtok", got, ref, TOL["bf16"])


# V, d, heads, head_dim, sigma: every instantiation, several slots with a short last one; sigma such that
# the scores spread by about one over the variables
COMMON = [(17, 512, 8, 64, 0.14), (40, 512, 16, 32, 0.14), (91, 1024, 16, 64, 0.1), (48, 1536, 8, 64, 0.08),
          (67, 2048, 16, 128, 0.07), (128, 2048, 8, 64, 0.07)]


@pytest.mark.parametrize("channels", [0, 4])
@pytest.mark.parametrize("s", [4, 16, 64, 256])
@pytest.mark.parametrize("V,d,H,dh,sigma", COMMON)
def test_agg_stream_common_component(lib, V, d, H, dh, sigma, s, channels):
    """Variables that share a component s times their spread (in every channel,
    or in a few large ones): the softmax does not see what it adds to all of a
    patch's scores, and neither may the token gradient, whose dS = a (dA - c)
    has it in dA and in c. A row sum c that is rounded apart from dA leaves
    2^-9 of it there: more than the usual bound from s = 16 on (all channels)
    or from s = 64 to 256 on (four)."""
    c, tok, prm, dz = _case(1, 6, V, d, H, dh, sigma)
    common = synth.normal(c.seed, "common", (1, 6, 1, d), dtype="bf16")
    if channels:
        common[..., channels:] = 0
    tok = synth.bf16_round(np.asarray(tok + s * common, np.float32))
    got, ref, a = _token_gradient(lib, tok, prm, dz, H, dh)
    assert 1.5 / V < a.max(-1).mean() < 0.9  # neither uniform weights nor single ones
    check("dtok", got, ref, TOL["bf16"])


@pytest.mark.parametrize("slot", [0, 1])
def test_agg_stream_infinite_scores(lib, slot):
    """Variables whose scores overflow to -inf weigh nothing, also when they
    fill the first slot of 16, before any finite score is known."""
    import torch
    from paper_2404_14712_amd._lib import AggDesc
    L, V, d, H, dh = 5, 40, 512, 8, 32
    _, tok, prm, _ = _case(1, L, V, d, H, dh, 0.1)
    # the query is all ones, so u_h[0] = 4 dh in every head
    prm["w_q"], prm["b_q"] = np.zeros_like(prm["w_q"]), np.ones_like(prm["b_q"])
    prm["w_k"][0] = 4.0
    tok[..., 0] = 0
    tok[:, :, 16 * slot:16 * slot + 16, 0] = synth.bf16_round(np.float32(-3e38))
    desc = AggDesc(1, L, V, d, H, dh, 1)
    z = torch.zeros(1, L, d, dtype=torch.bfloat16, device="cuda")
    saved = torch.full((lib.orbit_var_aggregate_saved_bytes(desc),), 255, dtype=torch.uint8, device="cuda")
    ws = torch.full((lib.orbit_var_aggregate_workspace_bytes(desc),), 255, dtype=torch.uint8, device="cuda")
    lib.orbit_var_aggregate(desc, dev(tok, "bf16"), {k: dev(v, "bf16") for k, v in prm.items()}, z, saved, ws)
    torch.cuda.synchronize()
    ref, cache = O.agg_fwd(tok, prm, H)
    assert cache["a"][..., 16 * slot:16 * slot + 16].max() == 0
    check("z", host(z), ref, TOL["bf16"])
