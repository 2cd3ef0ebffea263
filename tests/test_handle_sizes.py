"""Workspace sizes: a handle built for host queries alone gives the sizes that
the same problem needs on the device."""
import pytest

from paper_2605_07621_amd import ecut as E, inputs as I

# wide rings on the generic kernel (items cut into slices: one partial sum
# each), rows past the spin kernels', spin, spatial and up/down cuts
PROBLEMS = [I.Problem(I.xxz_chain(n, 1.0, 0.6, periodic=True), I.Cut("spatial", I.left_mask_first(cut)), k)
            for n, cut, k in [(33, 16, 1), (34, 17, 3), (36, 17, 4), (40, 20, 3), (24, 8, 12), (20, 4, 10), (12, 6, 6)]]
PROBLEMS += [I.Problem(I.hubbard_chain(10, 1.0, 3.0, V=0.7), I.Cut("spatial", I.left_mask_first(c)), 5, 4)
             for c in (2, 5, 8)]
PROBLEMS += [I.Problem(I.hubbard_chain(10, 1.0, 3.0), I.Cut("updn"), 5, 4)]
IDS = [f"{p.model.name}_{p.n_up}_{p.cut.left_mask}" for p in PROBLEMS]


def _up32(n):
    return (n + 31) // 32 * 32


@pytest.mark.parametrize("p", PROBLEMS[1:4], ids=IDS[1:4])
def test_host_only_workspace_holds_the_slices_partials(p):
    """Three vectors and one partial sum for every slice of the generic
    kernel's items: row tiles of max(longest row, 2048) amplitudes, cut into
    passes of 256 until a launch has about 4,096 groups."""
    S = E.Sectors.from_problem(p, host_only=True)
    b = S.blocks()
    tile = max(int(b[:, 3].max()), 2048)
    rows = [max(1, min(int(dl), tile // int(dr))) for dl, dr in b[:, 2:4]]
    n_items = sum(-(-int(dl) // r) for dl, r in zip(b[:, 2], rows))
    longest = max(r * int(dr) for r, dr in zip(rows, b[:, 3]))
    slices = n_items * max(1, min(-(-longest // 256), 4096 // n_items))
    assert slices > n_items
    assert S.lanczos_workspace(10) >= 3 * _up32(S.dim) + _up32(slices)


@pytest.mark.gpu
@pytest.mark.parametrize("p", PROBLEMS, ids=IDS)
def test_host_only_sizes_equal_the_device_handles(dev, p):
    host, device = E.Sectors.from_problem(p, host_only=True), E.Sectors.from_problem(p)
    for kw in (dict(), dict(reorth=True)):
        assert host.lanczos_workspace(40, **kw) == device.lanczos_workspace(40, **kw)
