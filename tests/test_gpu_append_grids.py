"""GPU: appends of more workgroups than one grid takes (2^32 threads), against the same groups in calls that fit one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


# one token of 8 channels: two workgroups of 256 threads per (frame, head) on the head_dim axis, three with a summary source of its own
@pytest.mark.parametrize("own_summary", (False, True))
def test_more_workgroups_than_a_grid(oqm, own_summary):
    H, d, F, part = 200, 8, 65535, 16384
    assert 2 * H * F > 2 ** 32 // 256 > 3 * H * part
    cfg = oqm.make_config(1, H, H, d, 1, 8, F, in_dtype=oqm.TOM_BF16, out_dtype=oqm.TOM_BF16)
    mems = [oqm.Memory.allocate(cfg) for _ in range(2)]
    try:
        g = torch.Generator(device="cuda").manual_seed(1)
        k, v, s = (torch.randn((F, 1, H, 1, d), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
        for m in mems:
            for t in (m.codes, m.meta, m.keys):
                t.zero_()
        oqm.tom_oqm_quantize_append(mems[0].handle, 0, 1, F, k, v, s if own_summary else None)
        for f in range(0, F, part):
            n = min(part, F - f)
            oqm.tom_oqm_quantize_append(mems[1].handle, 0, 1, n, k[f:], v[f:], s[f:] if own_summary else None)
        assert oqm.tom_oqm_num_groups(mems[0].handle) == oqm.tom_oqm_num_groups(mems[1].handle) == F
        for name in ("codes", "meta", "keys"):
            a, b = (getattr(m, name).view(torch.uint8) for m in mems)
            assert torch.equal(a, b) and a.any()
    finally:
        for m in mems:
            m.close()
