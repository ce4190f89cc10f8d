"""GPU: the group scores of the mean-query path against plain float64, on both sides of the rule that
folds the query inside the score kernel (short questions) or in a launch of its own."""
import pytest
import torch

pytestmark = pytest.mark.gpu

TDT = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


def _check(oqm, L, H, r, d, T, tq, dt, cosine, seed, scores_in_q=None):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    code = {"bf16": oqm.TOM_BF16, "f16": oqm.TOM_F16, "f32": oqm.TOM_F32}[dt]
    cfg = oqm.make_config(L, H, H * r, d, 1, 8, T, in_dtype=code, out_dtype=code,
                          sim=oqm.TOM_SIM_COSINE if cosine else oqm.TOM_SIM_DOT)
    mem = oqm.Memory.allocate(cfg)
    try:
        mem.keys.copy_(torch.randn(mem.keys.numel(), generator=gen, device="cuda").view_as(mem.keys))
        oqm.tom_oqm_set_num_groups(mem.handle, T)
        q = torch.randn((L, H * r, tq, d), generator=gen, device="cuda").to(TDT[dt])
        ws = torch.empty(oqm.tom_oqm_score_workspace_bytes(mem.handle, L, tq, oqm.TOM_SCORE_MEAN_QUERY, False),
                         dtype=torch.uint8, device="cuda")
        qb = q.double().view(L, H, r * tq, d).mean(2).reshape(L, 1, H * d).cpu()
        if scores_in_q is None:
            scores = torch.full((L, T + 3), 7.0, device="cuda")
        else:
            memory = q.view(-1).view(torch.float32)
            first = round(scores_in_q * (memory.numel() - L * (T + 3))) // 4 * 4
            scores = memory[first:first + L * (T + 3)].view(L, T + 3)
            between = scores[:, T:].clone()
        oqm.tom_oqm_score_groups(mem.handle, 0, L, q, tq, scores, T + 3, None, oqm.TOM_SCORE_MEAN_QUERY, ws)
        keys = mem.keys.double().view(L, T, H * d).cpu()
        want = (qb @ keys.transpose(1, 2))[:, 0]
        size = qb.norm(dim=-1) * keys.norm(dim=-1)
        # the mean's own terms are up to sqrt(r * T_q) larger than the mean: bound them by |q| / sqrt(r T_q) = 1
        slack = (size + keys.norm(dim=-1) * (H * d) ** 0.5) * 1e-14
        if cosine:
            want, slack = want / size.clamp_min(1e-24), slack / size.clamp_min(1e-24)
        got = scores[:, :T].double().cpu()
        assert ((got - want).abs() <= want.abs() * 2.0 ** -24 + slack).all()   # one rounding to float32
        assert torch.equal(scores[:, T:], torch.full_like(scores[:, T:], 7.0) if scores_in_q is None else between)
    finally:
        mem.close()


# d = 8 to 2048 (1 to 256 lanes per query row, idle lanes at 80 and 96); H_k * d under one batch of key
# loads (512), exactly one, several; one row slot per head (16 x 256) and none (the separate fold)
@pytest.mark.parametrize("H,r,d", ((1, 1, 8), (3, 2, 8), (4, 7, 128), (2, 1, 80), (5, 2, 80), (3, 4, 96), (8, 2, 256),
                                   (16, 1, 256), (1, 2, 2048), (4, 1, 2048), (64, 1, 128), (512, 1, 8)))
def test_head_shapes(oqm, H, r, d):
    for i, (T, tq) in enumerate(((1, 1), (31, 2), (32, 9), (33, 17))):
        _check(oqm, 2, H, r, d, T, tq, ("bf16", "f16", "f32")[i % 3], i % 2 == 0, 10 * d + i)


# 7 T_q rows in 8 slots, times (blocks + 168), against the rule's 3930 (float32 at this key: + 160, 3800), and 28 x 128 x T_q x (blocks + 64)
# against its 6.5e6: last fused and first separate question lengths
@pytest.mark.parametrize("L,T,tqs", ((1, 64, (26, 27)), (1, 256, (25, 26)), (8, 256, (18, 19)), (28, 256, (10, 11, 12)), (28, 1024, (1, 2))))
@pytest.mark.parametrize("dt", ("bf16", "f32"))
def test_both_sides_of_the_rule(oqm, L, T, tqs, dt):
    for tq in tqs:
        _check(oqm, L, 4, 7, 128, T, tq, dt, True, 1000 + tq)


# float32: two workgroups a compute unit (512) at keys of five pieces, one (256) above
@pytest.mark.parametrize("H,d", ((5, 64), (4, 80), (1, 328), (3, 128)))
def test_float32_rounds(oqm, H, d):
    for L, T in ((8, 1024), (8, 1025), (16, 1024), (16, 1025)):
        _check(oqm, L, H, 2, d, T, 2, "f32", L == 8, 3000 + d + T)


# float32 questions that an L2 holds beside an eighth of the keys, and of a token more
@pytest.mark.parametrize("L,T,tqs", ((28, 512, (20, 21)), (28, 256, (36, 37)), (14, 512, (40, 41)), (112, 128, (10, 11))))
def test_float32_past_l2(oqm, L, T, tqs):
    for tq in tqs:
        _check(oqm, L, 4, 4, 64, T, tq, "f32", True, 4000 + L + tq)


# scores written into the memory of the query: the query has to be consumed before the first of them
@pytest.mark.parametrize("where", (0.0, 0.5, 1.0))
@pytest.mark.parametrize("dt", ("bf16", "f32"))
def test_scores_in_the_memory_of_the_query(oqm, dt, where):
    for L, T, tq in ((1, 1000, 8), (2, 333, 16), (8, 256, 8)):
        _check(oqm, L, 4, 7, 128, T, tq, dt, True, 2000 + tq, scores_in_q=where)
