"""GPU parity of the reconstruction into float32, whose lanes take four channels each (eight above head_dim 1024).

Group sizes sit around four passes of 256 items (one workgroup per tile up to there, then equal chunks of at most
three passes) and at rows that leave the last pass or the last lanes of a pass idle.  Values are bit-exact against the oracle."""
import pytest
import torch

from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


@pytest.mark.parametrize("qaxis", (0, 1))
@pytest.mark.parametrize("d", (8, 24, 64, 72, 128, 520, 1016, 1024, 1032, 2048))
def test_float32_rows(oqm, d, qaxis):
    items = d // 4 if d <= 1024 else d // 8
    step = 256 // items * items if qaxis else 256
    sizes = sorted({max(1, p * step // items + o) for p in (1, 4, 6) for o in (-1, 0, 1)} | {1, 13})
    for i, G in enumerate(sizes):
        bits, meta = ((4, "f32"), (2, "bf16"), (4, "bf16"), (2, "f32"))[i % 4]
        st, mem = H.make_pair(oqm, n_layers=2, n_kv_heads=2, n_q_heads=2, head_dim=d, group_tokens=G, qgroup=8,
                              capacity=4, in_dtype=("f32", "bf16")[i % 2], out_dtype="f32", qaxis=qaxis, bits=bits, meta=meta)
        try:
            g = torch.Generator().manual_seed(100 * d + G)
            k, v = (torch.randn((4, 2, 2, G, d), generator=g).to(H.DT[("f32", "bf16")[i % 2]][1]) for _ in range(2))
            H.append_both(oqm, st, mem, k, v)
            q = torch.randn((2, 2, 2, d), generator=g)
            assert H.full_path_check(oqm, st, mem, q, 3)["k_eff"] == 3
        finally:
            mem.close()
