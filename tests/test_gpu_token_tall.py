"""GPU parity of the token-axis store of tiles that take workgroups of 512 or 1024 threads.

Tiles that 256 threads cannot hold in registers (13 rows of a lane at 16 bits, eight of float32; head_dim 64, 128 and 256 first go to the waves that hold a
tile): sizes at both sides of what 512 and 1024 threads hold, and past both, where the tile is read twice; head sizes whose rows leave threads idle, every code
width and metadata kind, with and without a summary source of its own.  Bit-exact against the oracle, summary keys within one float32 ulp."""
import pytest

from tests.test_gpu_token_rows import OPTS, _run, oqm  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ("bf16", "f16", "f32"))
@pytest.mark.parametrize("d", (72, 80, 128, 256, 520, 2048))
def test_tall_tiles(oqm, d, dt):  # noqa: F811
    rows = {threads: threads // (d // 8) * (8 if dt == "f32" else 13) for threads in (256, 512, 1024)}
    sizes = [r + o for r in rows.values() for o in (0, 1)] + [8 * (1024 // (d // 8)), rows[512] - 1]
    for i, G in enumerate(sorted(set(sizes))):
        bits, meta, sep = OPTS[(3 * i + d) % len(OPTS)]
        _run(oqm, d, G, dt, bits, meta, sep, 7000 + i, token_major=i % 2 == 1)


@pytest.mark.parametrize("bits, meta, sep", OPTS)
def test_options(oqm, bits, meta, sep):  # noqa: F811
    for dt, G in (("bf16", 196), ("bf16", 250), ("f32", 100), ("f32", 196)):
        _run(oqm, 256, G, dt, bits, meta, sep, 7100 + G)
