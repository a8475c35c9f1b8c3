"""GPU parity of the grouping of ragged batches at the edges of its chunks:
one workgroup counts and places 1024 systems a pass, and 256 workgroups share
a batch, so batches of 262144 and more take several passes each."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 1023, 1024, 1025, 262143, 262144, 262145, 300001])
@pytest.mark.parametrize("sizes", [(1, 4), (3, 3), (2, 32)])
def test_grouping_places_every_system(batch, sizes):
    """Diagonal systems of powers of two, so that x, ipiv and info are known
    exactly; every 97th size is refused with info = -1, its x left alone."""
    import paper_2609_15217_amd.lupp as L
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(batch)
    n = rng.integers(sizes[0], sizes[1] + 1, size=batch).astype(np.int32)
    bad = np.arange(batch) % 97 == 96
    offA, offB = np.cumsum(n.astype(np.int64) ** 2) - n.astype(np.int64) ** 2, np.cumsum(n.astype(np.int64)) - n
    A = np.zeros(int((n.astype(np.int64) ** 2).sum()))
    b = rng.integers(1, 1 << 20, size=int(n.sum())).astype(np.float64)
    row = np.arange(b.size) - np.repeat(offB, n)
    scale = 2.0 ** ((np.repeat(np.arange(batch), n) + row) % 5 - 2)
    A[np.repeat(offA, n) + row * (np.repeat(n, n) + 1)] = scale
    given = n.copy()
    given[bad] = np.where(np.arange(bad.sum()) % 2 == 0, 0, 33)
    t = [torch.from_numpy(v).to(dev) for v in (given, offA, offB, A, b)]
    ipiv = torch.zeros(b.size, dtype=torch.int32, device=dev)
    info = torch.full((batch,), -7, dtype=torch.int32, device=dev)
    ctx = L.Context(0)
    assert L.lupp_batched_solve_ragged(ctx, batch, *t, ipiv, info, L.LUPP_KEEP_A) == 0
    torch.cuda.synchronize()
    live = np.repeat(~bad, n)
    assert np.array_equal(info.cpu().numpy(), np.where(bad, -1, 0))
    assert np.array_equal(t[4].cpu().numpy(), np.where(live, b / scale, b))
    assert np.array_equal(ipiv.cpu().numpy(), np.where(live, row + 1, 0))
