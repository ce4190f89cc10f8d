"""GPU parity of the token-axis store kernels at every head_dim class and row count they split on.

The host takes head_dim 64, 128 and 256 to the form whose waves hold a tile in registers (8, 16 or
32 lanes per token row; 8, 4 or 2 rows per wave and pass; rows per lane in templates of 4, 6, 7, 8 and, for
16-bit inputs, 13; 1 to 4 waves); every other head_dim and a taller tile to the general form
(rows in registers up to 4 / 8 / 13 passes, read twice above).  A separate summary source has workgroups of its own in both.  Codes, scale / zero and
dequantized values are bit-exact against the oracle, summary keys within one float32 ulp."""
import pytest
import torch

from tests import harness as H

pytestmark = pytest.mark.gpu

TDT = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
OPTS = [(bits, meta, sep) for bits in (4, 2) for meta in ("f32", "bf16") for sep in (False, True)]


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


def _run(oqm, d, G, dt, bits, meta, sep, seed, token_major=False):
    st, mem = H.make_pair(oqm, n_layers=2, n_kv_heads=3, n_q_heads=3, head_dim=d, group_tokens=G, qgroup=8,
                          capacity=3, in_dtype=dt, qaxis=1, bits=bits, meta=meta)
    try:
        g = torch.Generator().manual_seed(seed)
        shape = (2, 2, G, 3, d) if token_major else (2, 2, 3, G, d)

        def draw():
            t = torch.randn(shape, generator=g).to(TDT[dt])
            return t.permute(0, 1, 3, 2, 4) if token_major else t
        k, v = draw(), draw()
        H.append_both(oqm, st, mem, k, v, draw() if sep else None)
        H.compare_storage(st, mem)
        q = torch.randn(2, 3, 2, d, generator=g).to(TDT[dt])
        assert H.full_path_check(oqm, st, mem, q, 2)["k_eff"] == 2
    finally:
        mem.close()


# rows per pass of one wave: 8, 4, 2; G as passes * rows (exact, one short, one over) at the
# template edges 4 | 6 | 7 | 8 rows with one wave, then two to four, 13 rows and the general form, without and with a
# summary source of its own.
@pytest.mark.parametrize("dt", ("bf16", "f16", "f32"))
@pytest.mark.parametrize("d", (64, 128, 256))
def test_tiles_held_by_row_waves(oqm, d, dt):
    per_pass = 512 // d
    passes = [0, 1, 4, 5, 6, 7, 8, 9, 13, 17, 24, 26, 32, 37, 39, 48, 52]
    sizes = sorted({max(1, p * per_pass + o) for p in passes for o in (-1, 0, 1)} | {50, 196 if d < 256 else 197})
    for i, G in enumerate(sizes):
        bits, meta, _ = OPTS[2 * i % len(OPTS)]
        _run(oqm, d, G, dt, bits, meta, False, 9000 + i, token_major=i % 3 == 1)
        if i % 3 == 0:
            _run(oqm, d, G, dt, bits, meta, True, 9050 + i, token_major=i % 2 == 1)
    for i, (bits, meta, sep) in enumerate(OPTS):   # every option at each template
        for p in (4, 6, 7, 8, 26 if d == 256 else 52):
            _run(oqm, d, p * per_pass, dt, bits, meta, False, 9200 + i)
            _run(oqm, d, p * per_pass - 1, dt, bits, meta, sep, 9100 + i)


# head_dim 96 (12 lanes per row, 21 rows per pass): 1, 5, 11 and 15 passes; 80 and 8 as spot checks
@pytest.mark.parametrize("dt", ("bf16", "f16", "f32"))
def test_general_form_at_other_head_dims(oqm, dt):
    for i, (bits, meta, sep) in enumerate(OPTS):
        for G in (16, 100, 230, 300):
            _run(oqm, 96, G, dt, bits, meta, sep, 9400 + i)
    _run(oqm, 80, 197, dt, 4, "f32", False, 9500)
    _run(oqm, 8, 50, dt, 4, "bf16", True, 9501)
