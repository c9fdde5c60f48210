"""Long rows that begin anywhere and end anywhere: the tiles of a streaming pass
begin on a 128-byte boundary of the row, what lies before and behind them goes
entry by entry.  The result is the k smallest (value, index) pairs, exactly."""
import pytest

pytestmark = pytest.mark.gpu

ROWS = 660   # one workgroup a row


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


@pytest.fixture(scope="module")
def h(torch):
    import paper_1309_5478_amd as knn
    return knn.Handle(0)


# a tile is 4096 entries: just above the on-chip rows, a whole number of tiles, one
# entry more and less, tiles that only fit without their head, short remainders
@pytest.mark.parametrize("cols", [16385, 20480, 20481, 20479, 20480 + 31, 24576 + 3, 40001])
@pytest.mark.parametrize("pad,begin", [(0, 0), (1, 0), (2, 1), (3, 5), (0, 31), (37, 2)])
def test_rows_of_any_alignment(h, torch, cols, pad, begin):
    print(f"select {ROWS}x{cols} pad {pad} begin {begin}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(cols * 100 + pad * 7 + begin)
    flat = torch.randint(0, 50000, (ROWS * (cols + pad) + begin,), generator=g, device="cuda").float()  # (ties)
    flat.mul_(0.37)
    x = flat[begin:begin + ROWS * (cols + pad)].view(ROWS, cols + pad)[:, :cols]
    x[::5, 3] = float("nan")
    x[::7, cols - 1] = float("-inf")
    x[1::7, 0] = -1.0
    want = torch.sort(x, dim=1, stable=True)   # (NaN last)
    for k in (1, 37, 300):
        for pivot in ("sample", "plain"):
            v, i = h.select_k(x, k, pivot=pivot)
            assert torch.equal(v, want[0][:, :k])
            assert torch.equal(i.long(), want[1][:, :k])
