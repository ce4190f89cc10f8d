"""GPU: the per-token scores of small launches against plain float64.

A launch of at most 512 units of 16 groups splits the contraction over the waves of a workgroup, with
1 to 4 tiles of 16 query tokens at a time (1 to 3 above 256 units); larger launches take the 64 x 64 form, unless few tokens meet long keys.  Most small ones
fold the query inside that launch, and so do the cases of the first tests here but for the largest. Scores that share memory with the question keep the
fold a launch of its own: the last tests ask the split form itself in this way.  The cases sit on
both sides of every edge: token tiles, group tiles, contractions that end in half a block of 16
channels or need several rounds of blocks, and the launch size itself."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


def _check(oqm, L, H, r, d, T, tq, cosine, seed, overlap=False):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    cfg = oqm.make_config(L, H, H * r, d, 1, 8, T, in_dtype=oqm.TOM_BF16, out_dtype=oqm.TOM_BF16,
                          sim=oqm.TOM_SIM_COSINE if cosine else oqm.TOM_SIM_DOT)
    mem = oqm.Memory.allocate(cfg)
    try:
        mem.keys.copy_(torch.randn(mem.keys.numel(), generator=gen, device="cuda").view_as(mem.keys))
        oqm.tom_oqm_set_num_groups(mem.handle, T)
        q = torch.randn((L, H * r, tq, d), generator=gen, device="cuda").to(torch.bfloat16)
        ws = torch.empty(oqm.tom_oqm_score_workspace_bytes(mem.handle, L, tq, oqm.TOM_SCORE_TOKEN_GEMM, True),
                         dtype=torch.uint8, device="cuda")
        qt = q.double().view(L, H, r, tq, d).mean(2).permute(0, 2, 1, 3).reshape(L, tq, H * d).cpu()
        if overlap:     # the scores go where the question is
            room = torch.full((max(q.numel() * 2 // 4, L * (T + 3)) + 4,), 7.0, device="cuda")
            inside = room.view(torch.bfloat16)[:q.numel()].view(q.shape)
            inside.copy_(q)
            q, scores = inside, room[:L * (T + 3)].view(L, T + 3)
        else:
            scores = torch.full((L, T + 3), 7.0, device="cuda")
        tok = torch.full((L * tq * T + 64,), 7.0, device="cuda")
        oqm.tom_oqm_score_groups(mem.handle, 0, L, q, tq, scores, T + 3, tok[:L * tq * T].view(L, tq, T),
                                 oqm.TOM_SCORE_TOKEN_GEMM, ws)
        keys = mem.keys.double().view(L, T, H * d).cpu()
        want = qt @ keys.transpose(1, 2)
        # one rounding to float32 (2^-24) on sums whose float64 error is far below the absolute term
        size = qt.norm(dim=-1)[:, :, None] * keys.norm(dim=-1)[:, None, :]
        got = tok[:L * tq * T].view(L, tq, T).double().cpu()
        assert ((got - want).abs() <= want.abs() * 2.0 ** -24 + size * 1e-14).all()
        group = want.mean(1)
        if cosine:
            group = group / (qt.mean(1).norm(dim=-1)[:, None].clamp_min(1e-12) * keys.norm(dim=-1).clamp_min(1e-12))
        slack = size.max(1).values if not cosine else torch.ones_like(group)
        got = scores[:, :T].double().cpu()
        assert ((got - group).abs() <= group.abs() * 2.0 ** -24 + slack * 1e-13).all()
        assert (overlap or (scores[:, T:] == 7.0).all()) and (tok[L * tq * T:] == 7.0).all()   # nothing outside the outputs
    finally:
        mem.close()


@pytest.mark.parametrize("tq", (1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 130))
def test_query_tokens_at_the_tile_edges(oqm, tq):
    for i, T in enumerate((1, 15, 16, 17, 50)):
        _check(oqm, 2, 2, 3, 64, T, tq, i % 2 == 0, 100 * tq + T)


# H_k * d = 8, 24: half a block; 128, 136: one block per wave and one more; 256, 264, 512, 520, 1032: rounds of two
@pytest.mark.parametrize("H,d", ((1, 8), (3, 8), (1, 128), (17, 8), (2, 128), (33, 8), (4, 128), (65, 8), (1, 1032)))
def test_contraction_lengths(oqm, H, d):
    for tq in (5, 40):
        _check(oqm, 1, H, 2, d, 37, tq, tq == 5, H * d + tq)


@pytest.mark.parametrize("L,T", ((1, 8192), (1, 8193), (16, 512), (16, 513), (512, 16), (513, 16), (57, 129)))
def test_launch_size_of_the_split_form(oqm, L, T):
    _check(oqm, L, 1, 1, 16, T, 3, True, L + T)


# above 256 units: 3 tiles in one pass; 4 (two passes of 2), 5, 6 and 7 (2 x 3, 3 x 3) and 10 tiles (4 x 3) with idle ones
@pytest.mark.parametrize("tq", (48, 49, 65, 96, 97, 145))
def test_passes_above_256_units(oqm, tq):
    for T in (4096, 4097):
        _check(oqm, 1, 1, 1, 24, T, tq, T == 4096, tq + T)


# The split form itself.  Tiles of a pass: one to four up to 256 units, up to three above; channels: half a block alone, half a block behind whole ones, fewer blocks than
# waves, one a wave and a half more, rounds of two and a rest.
@pytest.mark.parametrize("tq", (1, 16, 17, 33, 48, 49, 64, 65, 113, 130))
@pytest.mark.parametrize("H, d", ((1, 8), (3, 8), (1, 72), (1, 128), (17, 8), (33, 8), (65, 8)))
def test_split_form_at_the_tile_edges(oqm, H, d, tq):
    for i, T in enumerate((1, 15, 16, 17)):
        _check(oqm, 2, H, 1 + i % 2, d, T, tq, i % 2 == 0, 10 * tq + T, overlap=True)


@pytest.mark.parametrize("L, T", ((1, 4096), (1, 4097), (16, 512), (16, 513), (1, 8191), (3, 2720), (3, 2721)))   # 256 and 257, 512 and 528, 512, 510 and 513 units
def test_split_form_at_the_launch_sizes(oqm, L, T):
    for H, d, tq in ((1, 24, 3), (1, 40, 33), (3, 8, 49), (5, 24, 64), (1, 24, 97)):
        _check(oqm, L, H, 1, d, T, tq, tq % 2 == 0, L + T + tq, overlap=True)


# beyond 512 units, few tokens on long keys that end in half a block
@pytest.mark.parametrize("H, d, tq", ((1, 264, 8), (1, 264, 9), (65, 8, 16), (65, 8, 20), (65, 8, 26), (65, 8, 36)))
def test_split_form_of_long_keys(oqm, H, d, tq):
    for T in (9600, 9601):
        _check(oqm, 1, H, 3, d, T, tq, T == 9600, H + T + tq)
