"""Ragged batches by the number of work items: workgroups that take one item,
several, and batches of more items than one launch holds. The uniform solve of
the same systems gives the expected bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

ONE_PER = 65536       # up to here one workgroup per possible item
PER_LAUNCH = 1 << 23  # items of one launch


@pytest.fixture(scope="module")
def L():
    import paper_2609_15217_amd.lupp as L
    return L


def ragged(L, ctx, n, seed):
    """Solve N(0, 1) systems of sizes n (int32, device); compare every size
    with the uniform solve."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n64 = n.long()
    offA = torch.cumsum(n64 * n64, 0) - n64 * n64
    offB = torch.cumsum(n64, 0) - n64
    A = torch.randn(int((n64 * n64).sum()), generator=g, dtype=torch.float64, device="cuda")
    b = torch.randn(int(n64.sum()), generator=g, dtype=torch.float64, device="cuda")
    A0, b0 = A.clone(), b.clone()
    ipiv = torch.zeros(b.numel(), dtype=torch.int32, device="cuda")
    info = torch.full((n.numel(),), -7, dtype=torch.int32, device="cuda")
    assert L.lupp_batched_solve_ragged(ctx, n.numel(), n, offA, offB, A, b, ipiv, info, 0) == 0
    for m in torch.unique(n).tolist():
        at = torch.nonzero(n == m).flatten()
        ia = offA[at][:, None] + torch.arange(m * m, device="cuda")
        ib = offB[at][:, None] + torch.arange(m, device="cuda")
        uA, ub = A0[ia].contiguous(), b0[ib].contiguous()
        up = torch.zeros((at.numel(), m), dtype=torch.int32, device="cuda")
        ui = torch.zeros(at.numel(), dtype=torch.int32, device="cuda")
        assert L.lupp_batched_solve(ctx, m, at.numel(), L.LUPP_AOS, uA, m, m * m, ub, m, up, ui, 0) == 0
        assert torch.equal(info[at], ui)
        assert torch.equal(ipiv[ib], up)
        assert torch.equal(A[ia].view(torch.int64), uA.view(torch.int64))
        assert torch.equal(b[ib].view(torch.int64), ub.view(torch.int64))


@pytest.mark.parametrize("items", [ONE_PER, ONE_PER + 1, 2 * ONE_PER + 3])
def test_around_the_grid_rule(L, items):
    """n = 9 with 16 lanes: 16 systems per item, and 16 items more than those
    in the bound of its class; the last item is not full."""
    ctx = L.Context(0)
    assert L.lupp_set_ragged_lanes(ctx, 9, 16) == 0
    for bound in (items - 16, items):
        n = torch.full((16 * bound - 5,), 9, dtype=torch.int32, device="cuda")
        ragged(L, ctx, n, seed=items)


@pytest.mark.parametrize("sizes", [(22, 25), (17, 18, 21), (1, 2, 3, 5, 8, 13, 16), (2, 16, 17, 32)])
def test_several_items_per_workgroup(L, sizes):
    ctx = L.Context(0)
    # more possible items than ONE_PER in the classes of these sizes
    batch = 1_200_001 if max(sizes) > 16 else 2_300_001
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(sizes))
    pick = torch.randint(0, len(sizes), (batch,), generator=g, device="cuda")
    ragged(L, ctx, torch.tensor(sizes, dtype=torch.int32, device="cuda")[pick], seed=len(sizes))


def test_more_items_than_one_launch_holds(L):
    """2^23 items of 16 systems and some more: every system reads the same
    matrix (solve-only calls do not write it)."""
    m, batch = 9, 16 * PER_LAUNCH + 1003
    ctx = L.Context(0)
    assert L.lupp_set_ragged_lanes(ctx, m, 16) == 0
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    A = torch.randn((1, m * m), generator=g, dtype=torch.float64, device="cuda")
    b0 = torch.randn((1, m), generator=g, dtype=torch.float64, device="cuda")
    n = torch.full((batch,), m, dtype=torch.int32, device="cuda")
    offA = torch.zeros(batch, dtype=torch.int64, device="cuda")
    offB = torch.arange(batch, dtype=torch.int64, device="cuda") * m
    b = b0.expand(batch, m).contiguous()
    ipiv = torch.zeros((batch, m), dtype=torch.int32, device="cuda")
    info = torch.full((batch,), -7, dtype=torch.int32, device="cuda")
    assert L.lupp_batched_solve_ragged(ctx, batch, n, offA, offB, A, b, ipiv, info, L.LUPP_KEEP_A) == 0
    x, p = b0.clone(), torch.zeros((1, m), dtype=torch.int32, device="cuda")
    i = torch.zeros(1, dtype=torch.int32, device="cuda")
    assert L.lupp_batched_solve(ctx, m, 1, L.LUPP_AOS, A, m, m * m, x, m, p, i, L.LUPP_KEEP_A) == 0
    assert int(i) == 0 and bool((info == 0).all())
    assert bool((b == x).all())
    assert bool((ipiv == p).all())
