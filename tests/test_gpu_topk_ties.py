"""GPU: top-k in index order over rows in which scores repeat, against a stable sort.

The search counts eight bits at a time, lists the range of the k-th score once it holds
at most 16 of them, and compares a larger one that a digit has not divided with one of its scores.  The rows
sit on both sides of these: runs of 15 to 18 and of 65 equal scores, neighbours that differ in the last bits, one value
only, few values, both zeros and infinities, and sizes at the edges of the wave forms."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oqm():
    from paper_2510_18269_amd import oqm as m      # raises if the library is not built
    assert torch.cuda.is_available()
    return m


def _row(kind, n, g):
    x = torch.randn(n, generator=g)
    if kind == "distinct":
        return x
    if kind == "equal":
        return torch.full((n,), 0.25)
    if kind == "last bits":       # neighbours of 0.7 in float32
        return (torch.full((n,), 0.7).view(torch.int32) + torch.randint(0, 3, (n,), generator=g, dtype=torch.int32)).view(torch.float32)
    if kind == "zeros":
        x = torch.where(x > 0, 0.0, -0.0)
        x[n // 3], x[n // 2] = float("inf"), float("-inf")
        return x
    if kind == "negative":
        return -torch.pow(10.0, torch.randint(-38, 38, (n,), generator=g).float())
    if kind == "sorted":
        return x.sort().values
    copies = kind                 # every score that often, in random places
    return x[:(n + copies - 1) // copies].repeat(copies)[:n][torch.randperm(n, generator=g)]


KINDS = ("distinct", "equal", "last bits", "zeros", "negative", "sorted", 2, 5, 15, 16, 17, 18, 65, 200)


@pytest.mark.parametrize("n", (2, 64, 255, 256, 257, 320, 777, 1023, 1024, 1025, 2048, 3600, 4095, 4096))
def test_repeated_scores(oqm, n):
    g = torch.Generator().manual_seed(n)
    rows = torch.stack([_row(kind, n, g) for kind in KINDS])
    device = torch.full((len(KINDS), n + 3), 9.0, device="cuda")
    device[:, :n] = rows.cuda()
    order = torch.sort(rows + 0.0, dim=1, descending=True, stable=True).indices   # -0 + 0 = +0: equal scores, lowest index first
    for k in sorted({1, 2, 5, 63, 64, 65, n // 3, n // 2, n - 1, n}):
        if not 1 <= k <= n:
            continue
        idx = torch.full((len(KINDS), k), -7, dtype=torch.int32, device="cuda")
        assert oqm.tom_oqm_topk(device, n + 3, len(KINDS), n, k, idx) == k
        assert torch.equal(idx.cpu().long(), order[:, :k].sort(dim=1).values), k
