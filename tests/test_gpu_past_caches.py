"""GPU: calls that read past the caches (gathers that read more than 210 MB, keys of 100 MB and more) against the same work in
calls below those sizes: every bit equal."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


# tiles of one workgroup (four passes) and in chunks of three
@pytest.mark.parametrize("G", (50, 100))
@pytest.mark.parametrize("meta", ("f32", "bf16"))
@pytest.mark.parametrize("dt", ("bf16", "f16"))
def test_large_gather(oqm, dt, meta, G):
    L, H, d, T = 8, 4, 128, 64
    code, tdt = {"bf16": (oqm.TOM_BF16, torch.bfloat16), "f16": (oqm.TOM_F16, torch.float16)}[dt]
    k = 210_000_000 // (2 * L * H * G * (d // 2 + d // 64 * (4 if meta == "bf16" else 8))) + 1
    cfg = oqm.make_config(L, H, H, d, G, 64, T, in_dtype=code, out_dtype=code,
                          meta_dtype=oqm.TOM_BF16 if meta == "bf16" else oqm.TOM_F32)
    mem = oqm.Memory.allocate(cfg)
    g = torch.Generator(device="cuda").manual_seed(G)
    kv = [torch.randn((T, L, H, G, d), generator=g, device="cuda").to(tdt) for _ in range(2)]
    oqm.tom_oqm_quantize_append(mem.handle, 0, L, T, *kv)
    idx = torch.randint(0, T, (L, k), generator=g, device="cuda", dtype=torch.int32)
    whole = [torch.zeros((L, H, k * G, d), dtype=tdt, device="cuda") for _ in range(2)]
    oqm.tom_oqm_dequant_gather(mem.handle, 0, L, idx, k, k, *whole)
    for l in range(L):
        part = [torch.zeros((1, H, k * G, d), dtype=tdt, device="cuda") for _ in range(2)]
        oqm.tom_oqm_dequant_gather(mem.handle, l, 1, idx[l:l + 1].contiguous(), k, k, *part)
        assert all(torch.equal(w[l].view(torch.int16), p[0].view(torch.int16)) for w, p in zip(whole, part))
    mem.close()


# keys of one trip, whole and with a rest; of equal trips; of 512-byte pieces
@pytest.mark.parametrize("H,d", ((4, 128), (3, 96), (5, 128), (65, 8), (8, 128)))
def test_many_keys(oqm, H, d):
    L = 4
    T = 100_000_000 // (L * H * d * 4) + 1
    cfg = oqm.make_config(L, H, H, d, 1, 8, T, in_dtype=oqm.TOM_BF16, out_dtype=oqm.TOM_BF16, sim=oqm.TOM_SIM_COSINE)
    mem = oqm.Memory.allocate(cfg)
    g = torch.Generator(device="cuda").manual_seed(H * d)
    mem.keys.copy_(torch.randn(mem.keys.numel(), generator=g, device="cuda").view_as(mem.keys))
    oqm.tom_oqm_set_num_groups(mem.handle, T)
    q = torch.randn((L, H, 64, d), generator=g, device="cuda").to(torch.bfloat16)
    ws = torch.empty(oqm.tom_oqm_score_workspace_bytes(mem.handle, L, 64, oqm.TOM_SCORE_MEAN_QUERY, False), dtype=torch.uint8, device="cuda")
    scores, part = torch.zeros((L, T), device="cuda"), torch.zeros((1, T), device="cuda")
    oqm.tom_oqm_score_groups(mem.handle, 0, L, q, 64, scores, T, None, oqm.TOM_SCORE_MEAN_QUERY, ws)
    for l in range(L):
        oqm.tom_oqm_score_groups(mem.handle, l, 1, q[l:l + 1].contiguous(), 64, part, T, None, oqm.TOM_SCORE_MEAN_QUERY, ws)
        assert torch.equal(scores[l], part[0])
    mem.close()
