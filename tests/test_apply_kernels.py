"""Which kernels an application runs: the selection by size and tuning, from
the host tables alone."""
import pytest

from paper_2605_07621_amd import ecut as E, inputs as I


def _hub(n, a, b, ring=False):
    return I.Problem(I.hubbard_chain(n, 1.0, 4.0, periodic=ring), I.Cut("updn"), a, b)


def _spin(n, cut, k, ring=False):
    return I.Problem(I.xxz_chain(n, 1.0, 0.8, periodic=ring), I.Cut("spatial", I.left_mask_first(cut)), k)


def _ext(n, cut, a, b):
    return I.Problem(I.hubbard_chain(n, 1.0, 4.0, V=1.0), I.Cut("spatial", I.left_mask_first(cut)), a, b)


@pytest.mark.parametrize("p,want", [
    (_spin(16, 8, 8), "k_flat"), (_spin(24, 12, 12), "k_spinL+k_spinR"), (_spin(24, 8, 12), "k_spinL+k_spinR"),
    (_spin(28, 12, 9), "k_rows"), (_spin(36, 17, 3, ring=True), "k_rows"),
    (_spin(23, 16, 11), "k_spin"), (_spin(24, 16, 9), "k_spinL+k_spinR"), (_spin(24, 16, 12), "k_spinL+k_spinR"),
    (_ext(10, 5, 5, 5), "k_flat"), (_ext(14, 7, 7, 7), "k_spinL+k_spinR"), (_ext(16, 8, 5, 5), "k_rows"),
    (_ext(13, 7, 6, 6), "k_spinL+k_spinR"), (_ext(13, 7, 5, 5), "k_rows"), (_ext(13, 8, 6, 6), "k_rows"),
    (_ext(13, 10, 6, 6), "k_rows"),
    (_hub(12, 6, 6), "k_hubF"), (_hub(13, 6, 7, ring=True), "k_hubU+k_hubD"), (_hub(14, 7, 7), "k_hubP+k_hubD"),
    (_hub(16, 8, 8), "k_hubP+k_hub3"),
    (_hub(15, 7, 1), "k_hubF"), (_hub(16, 8, 1), "k_hub3"), (_hub(16, 8, 0), "k_hub3"), (_hub(16, 1, 8), "k_hubF"),
    (_hub(16, 8, 1, ring=True), "k_hub2"), (_hub(18, 9, 1), "k_hub2"), (_hub(20, 10, 1), "k_hub2"),
    (_hub(20, 10, 19), "k_hub2"), (_hub(16, 8, 2), "k_hubU+k_hubD"),
    (_hub(14, 7, 6), "k_hubU+k_hubD"), (_hub(15, 7, 7), "k_hubP+k_hub3"), (_hub(15, 7, 5), "k_hubP+k_hubD"), (_hub(15, 6, 7), "k_hubU+k_hub3"), (_hub(15, 5, 7), "k_hubU+k_hubD"),
    (_hub(16, 6, 6), "k_hubP+k_hub3"), (_hub(16, 5, 8), "k_hubU+k_hub3"), (_hub(16, 4, 8), "k_hubU+k_hub3"),
    (_hub(16, 3, 8), "k_hubU+k_hubD"), (_hub(17, 8, 4), "k_hubP+k_hubD"), (_hub(17, 6, 4), "k_hubU+k_hubD"),
    (_hub(18, 9, 3), "k_hubU+k_hubD")],
    ids=lambda v: v if isinstance(v, str) else f"{v.model.name}_{v.n_up}_{v.n_dn}_{v.cut.left_mask}")
def test_default_kernels(p, want):
    assert E.Sectors.from_problem(p, host_only=True).apply_kernels() == want


def test_kernels_of_named_variants():
    """A tuning that names a launch shape runs the kernels the shape belongs
    to, at every size; variant 6 alone leaves the choice to the library."""
    S = E.Sectors.from_problem(_hub(10, 5, 5), host_only=True)
    S.set_tuning(variant=6)
    assert S.apply_kernels() == "k_hubF"
    for t in (dict(grid=4), dict(tile=1), dict(n_xcd=8), dict(n_xcd=1), dict(row_order=1)):
        S.set_tuning(variant=6, **t)
        assert S.apply_kernels() == "k_hubU+k_hubD", t
    S = E.Sectors.from_problem(_hub(16, 8, 8), host_only=True)
    for v, want in ((1, "k_hub"), (2, "k_hub2"), (3, "k_upslab+k_hub3"), (4, "k_hubrow"), (5, "k_hubseg")):
        S.set_tuning(variant=v, n_xcd=8)
        assert S.apply_kernels() == want
    S = E.Sectors.from_problem(_hub(16, 8, 8), host_only=True)
    for t, want in ((dict(variant=6), "k_hubP+k_hubD"), (dict(variant=6, n_xcd=8, tile=8), "k_hubP+k_hubD"),
                    (dict(variant=6, grid=4), "k_hubU+k_hubD"), (dict(variant=6, n_xcd=1), "k_hubU+k_hubD"),
                    (dict(variant=7, n_xcd=8, row_order=8), "k_hubP+k_hub3"), (dict(variant=7, grid=8), "k_hubU+k_hub3"),
                    (dict(variant=7, tile=2), "k_hubU+k_hub3"), (dict(variant=7, n_xcd=1), "k_hubU+k_hub3")):
        S.set_tuning(**t)
        assert S.apply_kernels() == want, t
    S = E.Sectors.from_problem(_spin(24, 12, 12), host_only=True)
    for t, want in ((dict(tile=512), "k_spin"), (dict(variant=1), "k_rows"), (dict(variant=2), "k_spinL+k_spinR")):
        S.set_tuning(**t)
        assert S.apply_kernels() == want
