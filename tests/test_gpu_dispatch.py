"""Which kernel a solve runs (lupp_get_solve_kernel): the dispatcher's rules,
entries the caller set, and entries the autotuner measured."""
import pytest
import torch

from workloads import aos_to_soa, systems

pytestmark = pytest.mark.gpu

LARGE = 32768


@pytest.fixture(scope="module")
def L():
    import paper_2609_15217_amd.lupp as L
    return L


def autotune(L, ctx, n, layout, batch=LARGE):
    A, b, _ = systems(n, batch, seed=8200 + n)
    if layout == L.LUPP_SOA:
        A, b = aos_to_soa(A), aos_to_soa(b)
    tA, tb = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
    soa = layout == L.LUPP_SOA
    assert L.lupp_autotune(ctx, n, batch, layout, tA, n, batch if soa else n * n, tb,
                           batch if soa else n, reps=3)[0] == 0


@pytest.mark.parametrize("n,aos", [(12, True), (24, True), (20, False), (32, True)])
def test_autotuning_leaves_solve_only_calls_alone(L, n, aos):
    """The autotuner times calls that write the factors: solve-only calls keep
    the kernel they ran before, also where it cannot be forced."""
    ctx = L.Context(0)
    layout = L.LUPP_AOS if aos else L.LUPP_SOA
    before = L.lupp_get_solve_kernel(ctx, n, layout, LARGE, L.LUPP_KEEP_A)
    autotune(L, ctx, n, layout)
    assert L.lupp_get_solve_kernel(ctx, n, layout, LARGE, L.LUPP_KEEP_A) == before
    entry = L.lupp_get_dispatch(ctx, n, layout, LARGE)
    runs = L.lupp_get_solve_kernel(ctx, n, layout, LARGE)
    # with the factors: the entry, or the half-width kernel where that is faster
    assert runs == entry or (not aos and 17 <= n <= 24 and runs[1] == 8)
    # batches of the other size class were not timed
    other = L.Context(0)
    assert L.lupp_get_solve_kernel(ctx, n, layout, 100) == L.lupp_get_solve_kernel(other, n, layout, 100)


@pytest.mark.parametrize("n", [12, 20, 32])
def test_a_set_entry_serves_every_call(L, n):
    ctx = L.Context(0)
    entry = (L.LUPP_VARIANT_LANES, 16, 1)
    assert L.lupp_set_dispatch(ctx, n, L.LUPP_AOS, LARGE, *entry) == 0
    for flags in (0, L.LUPP_KEEP_A, L.LUPP_FMA):
        assert L.lupp_get_solve_kernel(ctx, n, L.LUPP_AOS, LARGE, flags) == entry
    assert L.lupp_set_pivoting(ctx, 4, 1e-10) == 0
    assert L.lupp_get_solve_kernel(ctx, n, L.LUPP_AOS, LARGE) == entry


def test_forced_variant_is_reported(L):
    ctx = L.Context(0)
    assert L.lupp_force_variant(ctx, L.LUPP_VARIANT_LANES, 32, 2) == 0
    assert L.lupp_get_solve_kernel(ctx, 20, L.LUPP_AOS, LARGE, L.LUPP_KEEP_A) == (2, 32, 2)
    with pytest.raises(L.LuppError):
        L.lupp_get_solve_kernel(ctx, 8, L.LUPP_AOS, LARGE)  # no 32-lane kernel of this size


@pytest.mark.parametrize("n,batch,kernel", [(5, 20000, (1, 1, 1)), (13, LARGE, (2, 8, 0))])
def test_interleaved_entries(L, n, batch, kernel):
    """Entries that measured faster over their whole size class than the one
    that won at the size the table was tuned at."""
    ctx = L.Context(0)
    for flags in (0, L.LUPP_KEEP_A):
        assert L.lupp_get_solve_kernel(ctx, n, L.LUPP_SOA, batch, flags) == kernel
