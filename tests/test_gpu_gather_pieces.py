"""The gather by 4 KB pieces of its output (large launches of the head_dim axis) against the gather by tiles, bit for bit.

Tiles of 1 to 12 pieces that are and are not whole waves, heads whose last round of pieces is whole, a part or a single piece, whole pieces or aligned, prefix rows that move the rows off a
piece's start, indices that name no stored group (their rows are left alone), repeated indices, and the one-call form that takes
every group in order and writes the indices.  The launches by tiles are small ones of the same groups, which the oracle covers
elsewhere; a launch above the line of the rule is large, hence the repeated groups.  And float32 tiles of the token axis, whose chunks
grow with the launch, the same way."""
import pytest
import torch

from tests import harness as H

pytestmark = pytest.mark.gpu

LINE = {"f32": 300_000_000, "bf16": 400_000_000, "f16": 400_000_000}


def line(out, G, d):
    """Bytes of output from which on the launch goes by pieces."""
    items = G * d // 8
    return LINE[out] if out == "f32" or items > 256 else 30_000_000 if items <= 208 else 170_000_000


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


def filled(oqm, L, heads, d, G, gs, T, out, bits, meta, seed, qaxis=0):
    code, dt = H.DT[out]
    cfg = oqm.make_config(L, heads, heads, d, G, gs, T, qaxis=qaxis, bits=bits, in_dtype=code, out_dtype=code,
                          meta_dtype=oqm.TOM_BF16 if meta == "bf16" else oqm.TOM_F32)
    mem = oqm.Memory.allocate(cfg)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    k, v = (torch.randn((T, L, heads, G, d), generator=gen, device="cuda").to(dt) for _ in range(2))
    oqm.tom_oqm_quantize_append(mem.handle, 0, L, T, k, v)
    return mem, dt


def by_tiles(oqm, mem, dt, L, heads, d, G, T):
    """Every group once: [L][heads][T][G][d] of K and V, a few groups to a launch."""
    parts = [[], []]
    step = max(1, 20_000_000 // (L * heads * G * d * 2 * dt.itemsize))
    for t in range(0, T, step):
        n = min(step, T - t)
        idx = torch.arange(t, t + n, dtype=torch.int32, device="cuda").repeat(L, 1)
        out = [torch.zeros((L, heads, n * G, d), dtype=dt, device="cuda") for _ in range(2)]
        oqm.tom_oqm_dequant_gather(mem.handle, 0, L, idx, n, n, *out)
        for p, o in zip(parts, out):
            p.append(o.view(L, heads, n, G, d))
    return [torch.cat(p, 2) for p in parts]


def raw(t):
    return t.view(torch.int16 if t.element_size() == 2 else torch.int32)


@pytest.mark.parametrize("G, d, gs, L, heads, prefix", (
    (4, 128, 8, 2, 2, 0),        # 64 items: one wave's
    (3, 176, 16, 3, 1, 0),       # 66
    (5, 104, 8, 1, 2, 1),        # 65
    (16, 104, 8, 2, 3, 3),       # 208
    (16, 128, 32, 2, 1, 0),      # one piece
    (50, 128, 64, 2, 3, 14),
    (61, 96, 32, 3, 1, 5),
    (196, 128, 64, 2, 1, 0),
    (37, 256, 128, 1, 2, 0),
    (13, 8, 8, 1, 2, 0),         # 13 items: stays with the tiles
))
@pytest.mark.parametrize("out, bits, meta", (("bf16", 4, "f32"), ("f16", 4, "bf16"), ("bf16", 2, "f32"), ("f16", 2, "bf16"), ("f32", 2, "f32"), ("f32", 2, "bf16")))
def test_pieces_against_tiles(oqm, G, d, gs, L, heads, prefix, out, bits, meta):
    T = 7
    mem, dt = filled(oqm, L, heads, d, G, gs, T, out, bits, meta, G * d)
    try:
        want = by_tiles(oqm, mem, dt, L, heads, d, G, T)
        group = 2 * L * heads * G * d * dt.itemsize
        k = line(out, G, d) // group + 3
        gen = torch.Generator(device="cuda").manual_seed(G)
        idx = torch.randint(-1, T + 1, (L, k), generator=gen, device="cuda", dtype=torch.int32)
        idx[:, -1], idx[:, 0] = T - 1, 0
        rows = prefix + k * G
        got = [torch.full((L, heads, rows, d), -3.0, dtype=dt, device="cuda") for _ in range(2)]
        if prefix:
            sys = [torch.randn((L, heads, prefix, d), generator=gen, device="cuda").to(dt) for _ in range(2)]
            oqm.tom_oqm_assemble_active(mem.handle, 0, L, idx, k, k, prefix, *sys, *got)
            for g, s in zip(got, sys):
                assert torch.equal(raw(g[:, :, :prefix].contiguous()), raw(s))
        else:
            oqm.tom_oqm_dequant_gather(mem.handle, 0, L, idx, k, k, *got)
        stored = (idx >= 0) & (idx < T)
        assert not bool(stored.all())
        for g, w in zip(got, want):
            for li in range(L):
                body = g[li, :, prefix:].view(heads, k, G, d)
                expect = w[li][:, idx[li].clamp(0, T - 1).long()]
                expect[:, ~stored[li]] = -3.0
                assert torch.equal(raw(body.contiguous()), raw(expect))
    finally:
        mem.close()


@pytest.mark.parametrize("prefix, off", ((0, 0), (14, 0), (0, 512), (3, 16)))
def test_last_round_of_a_head(oqm, prefix, off):
    """Whole rounds of 16 pieces and 1 to 15 left over, behind prefix rows and in buffers that start behind a piece's start."""
    L, heads, G, d, T = 2, 3, 49, 128, 5     # 3.06 pieces a tile
    mem, dt = filled(oqm, L, heads, d, G, 64, T, "bf16", 4, "f32", prefix + off)
    try:
        want = by_tiles(oqm, mem, dt, L, heads, d, G, T)
        gen = torch.Generator(device="cuda").manual_seed(prefix)
        k0 = line("bf16", G, d) // (2 * L * heads * G * d * 2) + 1
        left = set()
        for k in range(k0, k0 + 21):
            idx = torch.randint(0, T, (L, k), generator=gen, device="cuda", dtype=torch.int32)
            shape = (L, heads, prefix + k * G, d)
            n = L * heads * (prefix + k * G) * d
            room = [torch.full((n + off // 2 + 64,), -3.0, dtype=dt, device="cuda") for _ in range(2)]
            got = [r[off // 2:off // 2 + n].view(shape) for r in room]
            if prefix:
                sys = [torch.randn((L, heads, prefix, d), generator=gen, device="cuda").to(dt) for _ in range(2)]
                oqm.tom_oqm_assemble_active(mem.handle, 0, L, idx, k, k, prefix, *sys, *got)
                for g, s in zip(got, sys):
                    assert torch.equal(raw(g[:, :, :prefix].contiguous()), raw(s))
            else:
                oqm.tom_oqm_dequant_gather(mem.handle, 0, L, idx, k, k, *got)
            for r, g, w in zip(room, got, want):
                assert bool((r[:off // 2] == -3.0).all()) and bool((r[off // 2 + n:] == -3.0).all())
                for li in range(L):
                    assert torch.equal(raw(g[li, :, prefix:].view(heads, k, G, d)), raw(w[li][:, idx[li].long()]))
            left.add((k * G * d * 2 // 4096 + (k * G * d * 2 % 4096 > 0)) % 16)
        assert len(left) == 16
    finally:
        mem.close()


@pytest.mark.parametrize("G, d, gs, prefix, out, bits, meta", ((50, 128, 64, 0, "bf16", 4, "f32"), (61, 96, 32, 7, "f16", 4, "bf16"),
                                                              (33, 72, 8, 0, "bf16", 2, "f32"), (20, 128, 32, 3, "f32", 2, "f32")))
def test_every_group_in_order(oqm, G, d, gs, prefix, out, bits, meta):
    L, heads = 2, 2
    T = line(out, G, d) // (2 * L * heads * G * d * (4 if out == "f32" else 2)) + 2
    mem, dt = filled(oqm, L, heads, d, G, gs, T, out, bits, meta, G + d)
    try:
        want = by_tiles(oqm, mem, dt, L, heads, d, G, T)
        k, t_q = T + 3, 2                       # rows of the three absent groups are left alone
        gen = torch.Generator(device="cuda").manual_seed(G)
        q = torch.randn((L, heads, t_q, d), generator=gen, device="cuda").to(dt)
        sys = [torch.randn((L, heads, max(prefix, 1), d), generator=gen, device="cuda").to(dt) for _ in range(2)] if prefix else [None, None]
        ws = torch.empty(oqm.tom_oqm_score_workspace_bytes(mem.handle, L, t_q, oqm.TOM_SCORE_MEAN_QUERY, False), dtype=torch.uint8, device="cuda")
        scores = torch.zeros((L, T), dtype=torch.float32, device="cuda")
        idx = torch.full((L, k), -5, dtype=torch.int32, device="cuda")
        got = [torch.full((L, heads, prefix + k * G, d), -3.0, dtype=dt, device="cuda") for _ in range(2)]
        oqm.tom_oqm_retrieve(mem.handle, 0, L, q, t_q, k, scores, T, idx, *got, ws, path=oqm.TOM_SCORE_MEAN_QUERY,
                             prefix_rows=prefix, sys_k=sys[0], sys_v=sys[1])
        assert torch.equal(idx[:, :T], torch.arange(T, dtype=torch.int32, device="cuda").repeat(L, 1))
        for g, w, s in zip(got, want, sys):
            body = g[:, :, prefix:].reshape(L, heads, k, G, d)
            assert torch.equal(raw(body[:, :, :T].contiguous()), raw(w))
            assert bool((body[:, :, T:] == -3.0).all())
            if prefix:
                assert torch.equal(raw(g[:, :, :prefix].contiguous()), raw(s))
    finally:
        mem.close()


@pytest.mark.parametrize("G, d", ((33, 128), (50, 128), (61, 96), (80, 128), (81, 128)))   # 5, 7, 7, 10 and 11 passes
@pytest.mark.parametrize("bits, meta", ((4, "f32"), (2, "bf16")))
def test_large_float32_token_axis(oqm, G, d, bits, meta):
    """Tiles of up to ten passes go in chunks of four from 200 MB up, in chunks of three below."""
    L, heads, T = 2, 3, 5
    mem, dt = filled(oqm, L, heads, d, G, 8, T, "f32", bits, meta, G + d, qaxis=1)
    try:
        want = by_tiles(oqm, mem, dt, L, heads, d, G, T)
        k = 200_000_000 // (2 * L * heads * G * d * 4) + 1
        gen = torch.Generator(device="cuda").manual_seed(G)
        idx = torch.randint(0, T, (L, k), generator=gen, device="cuda", dtype=torch.int32)
        got = [torch.zeros((L, heads, k * G, d), dtype=dt, device="cuda") for _ in range(2)]
        oqm.tom_oqm_dequant_gather(mem.handle, 0, L, idx, k, k, *got)
        for g, w in zip(got, want):
            for li in range(L):
                assert torch.equal(raw(g[li].view(heads, k, G, d)), raw(w[li][:, idx[li].long()]))
    finally:
        mem.close()
