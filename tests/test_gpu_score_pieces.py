"""GPU: the group scores at every number of 64-channel pieces that a lane loads together, with and without a part of one
at the key's end, in both launches of the mean-query path, and the fold in parts of 64 channels with one, several and idle
row slots, against plain float64.  The helpers state the tolerance."""
import pytest
import torch

from tests.test_gpu_fused_fold import _check as check_mean
from tests.test_gpu_token_split import _check as check_tokens

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


# one to eight pieces of 64 channels, whole and with a rest; above 512 channels equal trips (640, 768, 896), eight pieces and a rest
# (520, 704), and from 1024 on pieces of 128 channels: 1024, 1152 (two trips and a rest), 1280, 2048, 2056
@pytest.mark.parametrize("H,d", ((1, 8), (1, 64), (1, 72), (2, 64), (1, 136), (3, 64), (1, 200), (2, 128), (2, 136), (3, 96), (5, 64),
                                 (3, 112), (3, 128), (7, 56), (7, 64), (4, 120), (4, 128), (65, 8), (5, 128), (11, 64), (6, 128), (7, 128),
                                 (8, 128), (9, 128), (5, 256), (8, 256), (257, 8)))
def test_pieces_of_the_key(oqm, H, d):
    for i, (L, T, tq) in enumerate(((2, 17, 3), (1, 70, 40))):
        check_mean(oqm, L, H, 2, d, T, tq, ("bf16", "f32")[i], True, H * d + i)
    # long questions, more rows than the rule allows a slot: fold and scores are launches of their own
    tq = 12 * max(1, 4096 // (H * d)) + 1
    check_mean(oqm, 1, H, 2, d, 33, tq, "f16", H % 2 == 0, H * d + 7)


# rows of a KV head (r * T_q) around the 64 slots of a part and the 512 rows of a trip, and around those of an undivided head
@pytest.mark.parametrize("d", (64, 80, 128, 192, 256))
def test_rows_of_the_fold(oqm, d):
    for r, tq in ((1, 63), (1, 64), (1, 65), (7, 9), (8, 64), (9, 57)):
        check_tokens(oqm, 2, 3, r, d, 21, tq, True, d + r * tq)
        check_tokens(oqm, 171, 3, r, d, 5, tq, True, d + r * tq + 1)     # 513 heads: whole, in 8, 16, 24 and 32 lanes a row
    check_mean(oqm, 600, 3, 8, d, 19, 64, "bf16", True, d)    # 64 + 600 workgroups: separate, one row more than a trip's
    check_mean(oqm, 600, 3, 8, d, 19, 65, "bf16", True, d + 1)
