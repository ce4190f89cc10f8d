"""The one-call retrieval of a small store: the gather's workgroups select their groups themselves."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


@pytest.mark.parametrize("T,k,L,G,dt,axis,prefix,where", [
    (2, 1, 1, 16, "bf16", 0, 0, "apart"), (64, 63, 2, 5, "f16", 0, 0, "apart"), (65, 64, 3, 7, "f32", 1, 9, "apart"),
    (255, 17, 1, 50, "bf16", 1, 0, "apart"), (256, 1, 2, 196, "bf16", 0, 3, "apart"), (256, 255, 1, 3, "f16", 0, 0, "apart"),
    (257, 20, 1, 16, "bf16", 0, 0, "apart"), (1023, 41, 2, 16, "f32", 1, 2, "apart"),      # four waves select
    (1024, 256, 1, 3, "f16", 0, 0, "apart"), (1024, 1, 1, 196, "bf16", 1, 0, "apart"),
    (1024, 257, 1, 3, "bf16", 0, 0, "apart"), (256, 128, 4, 16, "f16", 0, 0, "apart"),
    (1025, 20, 1, 16, "bf16", 0, 0, "apart"), (255, 129, 4, 16, "bf16", 0, 5, "apart"),    # one score too many; several rounds of workgroups
    (256, 128, 8, 16, "bf16", 0, 0, "apart"), (256, 129, 8, 16, "f16", 0, 3, "apart"),     # the most workgroups with one wave (4096), and one group more
    (256, 128, 16, 100, "bf16", 0, 0, "apart"), (256, 129, 16, 50, "f32", 1, 3, "apart"),  # the same where they make four passes (8192)
    (256, 128, 11, 70, "f16", 0, 0, "apart"), (256, 129, 11, 70, "bf16", 0, 0, "apart"),   # three passes (5632)
    (1000, 144, 2, 16, "bf16", 0, 0, "apart"), (1000, 145, 2, 16, "f16", 1, 0, "apart"),   # the same with four waves (1152, and 2048)
    (1000, 128, 4, 100, "f16", 1, 0, "apart"), (1000, 129, 4, 100, "bf16", 0, 0, "apart"),
    (100, 30, 2, 16, "bf16", 0, 0, "scores in k_out"), (100, 30, 2, 16, "bf16", 0, 0, "idx behind scores"),   # or shared memory (the second one only adjoins)
])
def test_retrieve_matches_separate_calls(oqm, T, k, L, G, dt, axis, prefix, where):
    _check(oqm, T, k, L, G, dt, axis, prefix, where)


@pytest.mark.parametrize("meta", ("f32", "bf16"))
@pytest.mark.parametrize("bits", (4, 2))
@pytest.mark.parametrize("dt", ("f32", "bf16", "f16"))
def test_every_form_of_the_selecting_gather(oqm, dt, bits, meta):
    """One and four selecting waves on both axes with three and four items a lane, and with five and seven where the token axis has 16-bit
    output (132 tiles).  Passes of a whole tile of 64 channels: one, two, four, five and seven at 16 bits; one, four and above,
    in chunks of three (token axis) or four, in float32.  Float32 items of eight channels, two to seven passes, above head_dim 1024."""
    for T in (200, 300):
        for G in (16, 60, 100, 150, 196):
            for axis in (0, 1):
                _check(oqm, T, 33, 1, G, dt, axis, 3, "apart", bits, meta)
        for G, axis in ((2, 0), (2, 1), (4, 1), (7, 0)) if dt == "f32" else ():
            _check(oqm, T, 33, 1, G, dt, axis, 3, "apart", bits, meta, d=1088)


def _check(oqm, T, k, L, G, dt, axis, prefix, where, bits=4, meta="f32", d=64):
    """Indices, scores and rows equal those of the separate calls bit for bit, with many equal scores."""
    H, tq, stride = 2, 3, T + 5
    code, tdt = {"f32": (oqm.TOM_F32, torch.float32), "bf16": (oqm.TOM_BF16, torch.bfloat16), "f16": (oqm.TOM_F16, torch.float16)}[dt]
    cfg = oqm.make_config(L, H, 4, d, G, 32, T, qaxis=axis, bits=bits, in_dtype=code, out_dtype=code,
                          meta_dtype=oqm.TOM_BF16 if meta == "bf16" else oqm.TOM_F32)
    mem = oqm.Memory.allocate(cfg)
    g = torch.Generator().manual_seed(T + k)
    kinds = torch.randint(0, max(2, T // 3), (T,), generator=g)      # repeated frames: equal scores, lowest index first
    kv = [torch.randn((int(kinds.max()) + 1, L, H, G, d), generator=g)[kinds].to(tdt).cuda() for _ in range(2)]
    oqm.tom_oqm_quantize_append(mem.handle, 0, L, T, *kv)
    q = torch.randn((L, 4, tq, d), generator=g).to(tdt).cuda()
    ws = torch.empty(oqm.tom_oqm_score_workspace_bytes(mem.handle, L, tq), dtype=torch.uint8, device="cuda")
    sys_kv = [torch.randn((L, H, prefix, d), generator=g).to(tdt).cuda() for _ in range(2)] if prefix else [None, None]
    rows = prefix + k * G

    def buffers():
        return (torch.full((L, stride), -9.0, device="cuda"), torch.full((L, k), -7, dtype=torch.int32, device="cuda"),
                *(torch.zeros((L, H, rows, d), dtype=tdt, device="cuda") for _ in range(2)))

    s0, i0, k0, v0 = buffers()
    oqm.tom_oqm_score_groups(mem.handle, 0, L, q, tq, s0, stride, None, oqm.TOM_SCORE_AUTO, ws)
    oqm.tom_oqm_topk(s0, stride, L, T, k, i0)
    oqm.tom_oqm_assemble_active(mem.handle, 0, L, i0, k, k, prefix, *sys_kv, k0, v0)
    s1, i1, k1, v1 = buffers()
    if where == "scores in k_out":
        s1 = k1.view(-1).view(torch.float32)[:L * stride].view(L, stride)
    elif where == "idx behind scores":
        s1 = torch.full((L * stride + L * k,), -9.0, device="cuda")
        i1 = s1[(L - 1) * stride + T - 3:].view(torch.int32)[3:3 + L * k].view(L, k)
        s1 = s1[:L * stride].view(L, stride)
    got = oqm.tom_oqm_retrieve(mem.handle, 0, L, q, tq, k, s1, stride, i1, k1, v1, ws, prefix_rows=prefix, sys_k=sys_kv[0], sys_v=sys_kv[1])
    torch.cuda.synchronize()
    assert got == k
    assert torch.equal(i0, i1)
    assert where == "scores in k_out" or torch.equal(s0[:, :T], s1[:, :T])
    assert torch.equal(k0.view(torch.uint8), k1.view(torch.uint8)) and torch.equal(v0.view(torch.uint8), v1.view(torch.uint8))
    mem.close()
