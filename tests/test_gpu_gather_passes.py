"""GPU parity of the reconstruction at every number of passes (of 256 items of 16 output bytes) that a workgroup takes.

A tile of up to four passes (token axis with 16-bit output: seven above 128 tiles, five above 2048) is one workgroup's, a taller one is cut into
equal chunks of at most three, four (head_dim axis with float32) or five (the token axis again).  Float32 output has items of four channels, of eight above
head_dim 1024.  Group sizes sit at both sides of each, with rows that leave the last pass or the last lanes of a
pass idle.  Values are bit-exact against the oracle."""
import pytest
import torch

from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


@pytest.mark.parametrize("out", ("f32", "bf16", "f16"))
@pytest.mark.parametrize("qaxis", (0, 1))
@pytest.mark.parametrize("d", (8, 24, 64, 72, 128, 520, 1016, 1024, 1032, 2048))
def test_passes_of_a_workgroup(oqm, d, qaxis, out):
    items = d // 4 if out == "f32" and d <= 1024 else d // 8
    step = 256 // items * items if qaxis else 256
    passes = (1, 4, 6, 8, 12) if out == "f32" else (1, 3, 4, 5, 6, 7, 8, 10, 13) if qaxis else (1, 3, 4, 6)
    sizes = sorted({max(1, p * step // items + o) for p in passes for o in (0, 1)} | {1, 13})
    layers = (2, 11) if qaxis and out != "f32" else (2,)      # 24 and 132 tiles
    shapes = [(G, L) for G in sizes for L in layers]
    if len(layers) > 1 and d in (72, 128):                    # 2052
        shapes += [(p * step // items, 171) for p in (5, 6, 7, 8)]
    for i, (G, L) in enumerate(shapes):
        bits, meta = ((4, "f32"), (2, "bf16"), (4, "bf16"), (2, "f32"))[(i + G) % 4]
        dt = ("f32", "bf16")[i % 2]
        st, mem = H.make_pair(oqm, n_layers=L, n_kv_heads=2, n_q_heads=2, head_dim=d, group_tokens=G, qgroup=8,
                              capacity=4, in_dtype=dt, out_dtype=out, qaxis=qaxis, bits=bits, meta=meta)
        try:
            g = torch.Generator().manual_seed(100 * d + G)
            k, v = (torch.randn((4, L, 2, G, d), generator=g).to(H.DT[dt][1]) for _ in range(2))
            H.append_both(oqm, st, mem, k, v)
            q = torch.randn((L, 2, 2, d), generator=g)
            assert H.full_path_check(oqm, st, mem, q, 3)["k_eff"] == 3
        finally:
            mem.close()
