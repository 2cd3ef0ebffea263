"""The entanglement spectrum's lanes (streams and eigensolver handles of the
library) beside the caller's own streams and memory."""
import numpy as np
import pytest

from paper_2605_07621_amd import ecut as E, inputs as I


@pytest.mark.gpu
def test_refused_while_the_stream_is_captured(dev):
    """A call inside a graph capture is refused, the capture goes on and its
    graph replays, and the library's lanes serve later calls: the same values
    bit for bit."""
    torch = pytest.importorskip("torch")
    p = I.Problem(I.hubbard_chain(8, 1.0, 4.0, V=0.5), I.Cut("spatial", I.left_mask_first(4)), 4, 4)
    s = E.Sectors.from_problem(p)
    x = torch.from_numpy(I.psi(17, s.dim)).to(dev)
    ref = np.concatenate(s.entanglement(x)["lam"])
    y = torch.zeros_like(x)
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        y.add_(x)
        with pytest.raises(E.EcutError):
            s.entanglement(x, stream=side)
        y.add_(x)
    for k in range(1, 4):
        g.replay()
        assert np.array_equal(np.concatenate(s.entanglement(x)["lam"]), ref)
        torch.cuda.synchronize()
        assert torch.equal(y, sum([x] * (2 * k - 1), x))


# (problem, the old single chain's workspace in words): the largest group of
# equal blocks, its off-diagonals, every eigenvalue, a status word a block
@pytest.mark.parametrize("p", [
    I.Problem(I.xxz_chain(12, 1.0, 0.7), I.Cut("spatial", I.left_mask_first(6)), 6),
    I.Problem(I.xxz_chain(30, 1.0, 0.7), I.Cut("spatial", I.left_mask_first(15)), 15),
    I.Problem(I.xxz_chain(31, 1.0, 0.7), I.Cut("spatial", I.left_mask_first(15)), 15),
    I.Problem(I.xxz_chain(32, 1.0, 0.7), I.Cut("spatial", I.left_mask_first(16)), 16),
    I.Problem(I.hubbard_chain(14, 1.0, 4.0, V=0.5), I.Cut("spatial", I.left_mask_first(7)), 7, 7)],
    ids=["spin12", "spin30", "spin31", "spin32", "hubbard14"])
def test_workspace_beside_the_largest_group_is_bounded(p):
    """The blocks that run side by side take at most 1 GiB (and their
    off-diagonals) more than the largest group of equal blocks alone."""
    import ctypes
    S = E.Sectors.from_problem(p, host_only=True)
    m = S.blocks()[:, 2:4].min(axis=1)
    sizes, counts = np.unique(m[m > 0], return_counts=True)
    one_chain = int(max(sizes * sizes * counts) + max(sizes * counts) + m.sum() + (len(m) + 1) // 2 + 1)
    nl = E._sz()
    got = int(E.lib().ecut_entanglement_sizes(S.h, ctypes.byref(nl)))
    assert nl.value == m.sum()
    assert one_chain <= got <= one_chain + (1 << 27) + m.sum()


# one chain on the caller's stream (one size; sizes of 11 and 42 rows
# together) and lanes of the library (64 rows, 163, 87)
@pytest.mark.gpu
@pytest.mark.parametrize("p", [
    I.Problem(I.hubbard_chain(6, 1.0, 4.0), I.Cut("updn"), 3, 3),
    I.Problem(I.xxz_chain(8, 1.0, 0.7), I.Cut("spatial", I.left_mask_first(4)), 4),
    I.Problem(I.xxz_chain(12, 1.0, 0.7), I.Cut("spatial", I.left_mask_first(6)), 6),
    I.Problem(I.xxz_chain(15, 1.0, 0.7), I.Cut("spatial", I.left_mask_first(7)), 7),
    I.Problem(I.xxz_chain(14, 1.0, 0.7), I.Cut("spatial", I.left_mask_first(7)), 7),
    I.Problem(I.xxz_chain(16, 1.0, 0.7), I.Cut("spatial", I.left_mask_first(8)), 8),
    I.Problem(I.hubbard_chain(8, 1.0, 4.0, V=0.5), I.Cut("spatial", I.left_mask_first(4)), 4, 4)],
    ids=["one_size", "11", "42", "64_odd", "64", "163", "87"])
def test_spectrum_on_one_chain_and_on_lanes(dev, p):
    """lambda of a random state against the squared singular values of its
    blocks in numpy (|d lambda| <= 1e-13: a Gram matrix's error is about eps
    times its largest eigenvalue, at most 1), on the default stream and, bit
    for bit the same, on another one right after work there."""
    torch = pytest.importorskip("torch")
    s = E.Sectors.from_problem(p)
    psi = I.psi(23, s.dim)
    psi /= np.linalg.norm(psi)
    x = torch.from_numpy(psi).to(dev)
    got = s.entanglement(x)
    for k, (_, _, dl, dr, off) in enumerate(s.blocks()):
        ref = np.linalg.svd(psi[off:off + dl * dr].reshape(dl, dr), compute_uv=False) ** 2
        assert np.max(np.abs(got["lam"][k] - ref)) <= 1e-13
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        again = s.entanglement(4.0 * (0.25 * x))
    for a, b in zip(got["lam"], again["lam"]):
        assert np.array_equal(a, b)
