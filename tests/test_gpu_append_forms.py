"""GPU parity of the head_dim-axis store in its two forms, at the edges where they differ.

A K tile is walked by one workgroup in trips of four rows per lane, or it is cut into chunks of two
rows per lane and its key made by workgroups of their own: for keys taken from another tensor, and
for small launches of tiles taller than one trip.  The keys' column sums are joined by lane swaps at 8, 16 and 32 lanes per row
and through LDS otherwise, in one part per 64 channels while the launch is small.  Tall tiles are walked by 1024 threads.  The workgroups that walk or
make keys stand in front of the last 6272 chunks, so larger launches have chunks on both sides.  Codes, scale / zero and dequantized
values are bit-exact against the oracle, summary keys within one float32 ulp."""
import pytest
import torch

from tests import harness as H

pytestmark = pytest.mark.gpu

TDT = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


def _run(oqm, *, d, G, frames, heads, dt="bf16", sep=False, bits=4, meta="f32", layers=1, gs=8, token_major=False, seed=0):
    st, mem = H.make_pair(oqm, n_layers=layers, n_kv_heads=heads, n_q_heads=heads, head_dim=d, group_tokens=G, qgroup=gs,
                          capacity=frames + 1, in_dtype=dt, bits=bits, meta=meta)
    try:
        g = torch.Generator().manual_seed(seed)

        def draw(n):
            t = torch.randn((n, layers, G, heads, d) if token_major else (n, layers, heads, G, d), generator=g).to(TDT[dt])
            return t.permute(0, 1, 3, 2, 4) if token_major else t
        for n in (1, frames):      # the second call does not start at group 0
            k, v = draw(n), draw(n)
            H.append_both(oqm, st, mem, k, v, draw(n) if sep else None)
        H.compare_storage(st, mem)
    finally:
        mem.close()


# lanes per row 1 (256 rows per pass), 3, 8, 12, 16, 24, 32, 64, 256 (one row per pass); G around one chunk (two passes), one trip (four)
@pytest.mark.parametrize("dt", ("bf16", "f16", "f32"))
@pytest.mark.parametrize("d", (8, 24, 64, 96, 128, 192, 256, 512, 2048))
def test_small_launches_at_the_edges_of_chunks_and_trips(oqm, d, dt):
    rpp = 256 // (d // 8)
    sizes = sorted({max(1, p * rpp + o) for p in (1, 2, 4, 8) for o in (-1, 0, 1)} | {1, 197})
    for i, G in enumerate(sizes):
        for sep in (False, True):
            _run(oqm, d=d, G=G, frames=2, heads=3, dt=dt, sep=sep, bits=(4, 2)[i % 2], meta=("f32", "bf16")[i // 2 % 2],
                 layers=2, token_major=i % 3 == 1, seed=100 * d + 2 * i + sep)


# tiles of the second call on both sides of the limits: 256 (float32), 384 (16-bit) and one workgroup per compute unit for the keys
@pytest.mark.parametrize("dt,frames", [(dt, f) for dt in ("bf16", "f32") for f in (42, 43, 63, 64, 65, 96, 97)])
def test_both_sides_of_the_rule(oqm, dt, frames):
    for sep in (False, True):
        _run(oqm, d=128, G=70, frames=frames, heads=2, dt=dt, sep=sep, gs=64, seed=frames)
    _run(oqm, d=64, G=130, frames=frames, heads=2, dt=dt, gs=32, seed=frames + 1)
    _run(oqm, d=80, G=101, frames=frames, heads=2, dt=dt, gs=16, seed=frames + 2)


# chunks of the second call below, at and above the 6272 that stand behind the walks and the keys
@pytest.mark.parametrize("frames,heads,G", [(392, 4, 65), (392, 8, 35), (393, 8, 35), (1000, 8, 33), (700, 8, 100)])
def test_chunks_on_both_sides_of_the_long_workgroups(oqm, frames, heads, G):
    for sep in (False, True):
        _run(oqm, d=128, G=G, frames=frames, heads=heads, sep=sep, gs=32, seed=frames + G)


# tiles just above 64 KB, 162 of K: walked by 1024 threads, two passes a chunk and four a trip.  G around both, with a rest that leaves waves idle
@pytest.mark.parametrize("dt", ("bf16", "f32"))
@pytest.mark.parametrize("d", (8, 24, 64, 96, 128, 192, 256, 512, 2048))
def test_tall_tiles(oqm, d, dt):
    rpp = 1024 // (d // 8)
    low = 65536 // (d * (2 if dt == "bf16" else 4))
    base = (low // (4 * rpp) + 1) * 4 * rpp
    for i, G in enumerate((base, base + 1) if dt == "bf16" else (base - 1 if base - 1 > low else base + 2 * rpp, base + 2 * rpp + 1)):
        _run(oqm, d=d, G=G, frames=81, heads=2, dt=dt, bits=(4, 2)[i], meta=("f32", "bf16")[i], token_major=i == 1, seed=d + i)


# above 96 KB at any number of tiles; fewer of them are cut
@pytest.mark.parametrize("frames,G", [(20, 390), (100, 390), (400, 520)])
def test_tiles_above_96_kb(oqm, frames, G):
    _run(oqm, d=128, G=G, frames=frames, heads=2, gs=64, seed=frames)
