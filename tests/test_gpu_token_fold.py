"""GPU: per-token scores of launches that fold the query inside the contraction, against plain float64.

fold_tiles decides by query heads per KV head, tokens, channels and launch size; the cases sit on both sides: one to nine query heads per KV head
(loaded one, two or four at a time, above that in turns), token tiles and passes, channels that end inside a block of 32 or inside a
lane's eight, heads whose width is no multiple of a block, few and many units, and, behind the line, the launch with a fold of its own."""
import pytest
import torch

from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


def _check(oqm, L, heads, r, d, T, tq, dtype="bf16", cosine=True, tokens=True, overlap=False):
    gen = torch.Generator(device="cuda").manual_seed(L + 10 * r + 100 * d + 1000 * T + tq)
    code, dt = H.DT[dtype]
    cfg = oqm.make_config(L, heads, heads * r, d, 1, 8, T, in_dtype=code, out_dtype=code,
                          sim=oqm.TOM_SIM_COSINE if cosine else oqm.TOM_SIM_DOT)
    mem = oqm.Memory.allocate(cfg)
    try:
        mem.keys.copy_(torch.randn(mem.keys.numel(), generator=gen, device="cuda").view_as(mem.keys))
        oqm.tom_oqm_set_num_groups(mem.handle, T)
        q = torch.randn((L, heads * r, tq, d), generator=gen, device="cuda").to(dt)
        qt = q.double().view(L, heads, r, tq, d).mean(2).permute(0, 2, 1, 3).reshape(L, tq, heads * d).cpu()
        ws = torch.empty(oqm.tom_oqm_score_workspace_bytes(mem.handle, L, tq, oqm.TOM_SCORE_TOKEN_GEMM, tokens),
                         dtype=torch.uint8, device="cuda")
        stride = T + 3
        if overlap:     # the scores go where the question is
            room = torch.zeros(max(q.numel() * q.element_size(), L * stride * 4) // 4 + 4, dtype=torch.float32, device="cuda")
            q2 = room.view(dt)[:q.numel()].view(q.shape)
            q2.copy_(q)
            q, scores = q2, room[:L * stride].view(L, stride)
        else:
            scores = torch.full((L, stride), 7.0, device="cuda")
        tok = torch.full((L * tq * T + 64,), 7.0, device="cuda")
        oqm.tom_oqm_score_groups(mem.handle, 0, L, q, tq, scores, stride, tok[:L * tq * T].view(L, tq, T) if tokens else None,
                                 oqm.TOM_SCORE_TOKEN_GEMM, ws)
        keys = mem.keys.double().view(L, T, heads * d).cpu()
        want = qt @ keys.transpose(1, 2)
        size = qt.norm(dim=-1)[:, :, None] * keys.norm(dim=-1)[:, None, :]
        if tokens:      # one rounding to float32 (2^-24) on sums whose float64 error is far below the absolute term
            got = tok[:L * tq * T].view(L, tq, T).double().cpu()
            assert ((got - want).abs() <= want.abs() * 2.0 ** -24 + size * 1e-14).all()
        assert (tok[L * tq * T if tokens else 0:] == 7.0).all()
        group = want.mean(1)
        if cosine:
            group = group / (qt.mean(1).norm(dim=-1)[:, None].clamp_min(1e-12) * keys.norm(dim=-1).clamp_min(1e-12))
        slack = size.max(1).values if not cosine else torch.ones_like(group)
        got = scores[:, :T].double().cpu()
        assert ((got - group).abs() <= group.abs() * 2.0 ** -24 + slack * 1e-13).all()
        if not overlap:
            assert (scores[:, T:] == 7.0).all()
    finally:
        mem.close()


@pytest.mark.parametrize("dtype", ("f32", "bf16", "f16"))
@pytest.mark.parametrize("r", (1, 2, 3, 4, 5, 7, 9))
def test_query_heads_and_types(oqm, r, dtype):
    for i, tq in enumerate((1, 16, 17, 33, 64, 65)):
        _check(oqm, 2, 2, r, (64, 40, 128)[i % 3], (17, 16, 50)[i % 3], tq, dtype, cosine=i % 2 == 0)


# channels: less than a lane's round, one block and a bit, whole blocks, one block a wave and one more, several rounds
@pytest.mark.parametrize("heads, d", ((1, 8), (3, 8), (5, 8), (1, 32), (3, 24), (1, 256), (33, 8), (3, 88), (5, 200), (1, 2048)))
def test_channels(oqm, heads, d):
    for r, tq in ((1, 20), (2, 1), (4, 48)):
        _check(oqm, 1, heads, r, d, 33, tq)


@pytest.mark.parametrize("L, T", ((1, 1), (1, 256 * 16), (1, 256 * 16 + 1), (8, 1024), (8, 1025), (4, 4400), (4, 4401)))
def test_launch_sizes(oqm, L, T):
    for r, tq in ((1, 16), (2, 33), (4, 45), (7, 16), (1, 70)):
        _check(oqm, L, 3, r, 64, T, tq, tokens=tq < 40)


def test_folds_of_their_own(oqm):
    for L, heads, r, d, T, tq, dtype in ((1, 4, 7, 128, 100, 64, "bf16"), (9, 4, 7, 128, 500, 33, "f16"), (1, 4, 7, 128, 40, 16, "f32"),
                                         (2, 8, 4, 256, 60, 1, "bf16"), (1, 2, 16, 1024, 40, 40, "bf16"), (1, 2, 1, 2048, 40, 5, "bf16")):
        _check(oqm, L, heads, r, d, T, tq, dtype)


def test_scores_over_the_question(oqm):
    for T, tq in ((40, 16), (700, 3)):
        _check(oqm, 2, 2, 2, 64, T, tq, overlap=True)


# one tile of tokens, launches beyond two rounds of the chip: the contraction is split or, at more tokens and units, 64 x 64
@pytest.mark.parametrize("tq, units", ((1, 1650), (8, 1300), (12, 1100), (16, 900)))
def test_one_tile_of_tokens_on_long_keys(oqm, tq, units):
    for heads, d, r, T in ((2, 128, 3, units // 10 * 16), (2, 128, 3, units // 10 * 16 + 1), (3, 80, 3, units // 10 * 16), (4, 136, 4, units // 10 * 16 - 5)):
        _check(oqm, 10, heads, r, d, T, tq, cosine=tq != 8)
    for T in ((2000 - 75 * tq) // 10 * 16, (2000 - 75 * tq) // 10 * 16 + 1):
        _check(oqm, 10, 4, 3, 256, T, tq, tokens=False)


# ... and both sides of its lines, which step with every 256 units of 16 groups and go by channels and tokens
@pytest.mark.parametrize("heads, d, units, tq", ((2, 128, 768, 8), (2, 128, 768, 9), (2, 128, 769, 1), (2, 128, 1025, 7), (2, 128, 1280, 8), (3, 96, 1024, 4), (3, 96, 1024, 5), (5, 80, 1536, 4), (5, 80, 1281, 5),
                                                 (4, 128, 1024, 7), (4, 128, 1024, 8), (4, 128, 1280, 12), (4, 128, 1281, 5), (4, 128, 1281, 6), (4, 256, 1792, 5), (4, 256, 1537, 6), (4, 256, 1793, 1), (4, 256, 1793, 2)))
def test_steps_of_one_tile(oqm, heads, d, units, tq):
    _check(oqm, 1, heads, 3, d, units * 16 - units % 3, tq, tokens=tq % 2 == 0, cosine=units % 2 == 0)


# the same units cut into 16 or 64 groups by short layers: 260 units of 64 step as 1025 of 16 do
def test_short_layers_of_one_tile(oqm):
    for T in (17, 65):
        _check(oqm, 260, 4, 2, 64, T, 2)


# two and three tiles whose last is mostly empty, where the 64 x 64 form would leave a third of one round idle, up to 168 units of 64, or, three tiles, two fifths of two, 257 to 308
@pytest.mark.parametrize("tq", (17, 25, 26, 33, 38, 39))
def test_nearly_empty_tiles_on_long_keys(oqm, tq):
    for i, T in enumerate((6 * 64, 6 * 64 + 1, 9 * 64, 9 * 64 + 1, 11 * 64, 11 * 64 + 1)):
        _check(oqm, 28, 4, 3, 128 + 8 * (i % 2), T, tq, tokens=i % 2 == 0, cosine=i != 2)


# units of 32 groups: from 257 units of 64 to 768 of 32, one, two or four token tiles in the last pass; launches on both sides
@pytest.mark.parametrize("tq", (17, 32, 33, 49, 64, 65, 96, 100, 130))
def test_units_of_32_groups(oqm, tq):
    for i, T in enumerate((25 * 64, 25 * 64 + 1, 26 * 64 - 31, 26 * 64 - 32, 76 * 32 - 1, 76 * 32, 76 * 32 + 1)):
        _check(oqm, 10, (5, 3)[i % 2], 3, (8, 40)[i % 2], T, tq, cosine=i % 3 != 0, tokens=i != 1)
