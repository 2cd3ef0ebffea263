"""Batched applications whose problems take different left passes, and the
default tuning just above the sizes where it changes kernel."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2605_07621_amd import ecut as E, inputs as I

pytestmark = pytest.mark.gpu


def _hub(n, a, b, ring=False, u=3.0):
    return I.Problem(I.hubbard_chain(n, 0.9, u, periodic=ring), I.Cut("updn"), a, b)


# one problem per kind of launch: (problem, tuning, kernels)
KINDS = {
    "fused": (_hub(9, 4, 5), {}, "k_hubF"),
    "general": (_hub(10, 5, 4, ring=True), dict(variant=6, n_xcd=8, tile=2), "k_hubU+k_hubD"),
    "general odd": (_hub(9, 4, 3), dict(variant=6, grid=8), "k_hubU+k_hubD"),
    "panels 14": (_hub(14, 6, 2), dict(variant=6, n_xcd=8), "k_hubP+k_hubD"),
    "panels 17": (_hub(17, 3, 2), dict(variant=6, n_xcd=8), "k_hubP+k_hubD"),
    "panels by default": (_hub(14, 7, 7), {}, "k_hubP+k_hubD"),
    "general by default": (_hub(13, 6, 5, ring=True), {}, "k_hubU+k_hubD"),
    "class tiles": (_hub(14, 5, 3), dict(variant=7, n_xcd=8), "k_hubP+k_hub3"),
    "spin": (I.Problem(I.xxz_chain(14, 1.0, 0.8), I.Cut("spatial", I.left_mask_first(7)), 7), {}, "k_flat"),
    "rows": (I.Problem(I.xxz_chain(34, 1.0, 0.6), I.Cut("spatial", I.left_mask_first(17)), 2), {}, "k_rows"),
}
BATCHES = [
    ["fused", "general", "panels 14", "general odd"],
    ["panels 14", "fused", "general odd", "panels 17", "general"],
    ["general", "panels 17", "panels 14"],
    ["panels 14", "panels 17"],                      # no item of the general left pass
    ["panels 17"],
    ["panels 14", "fused"],
    ["spin", "panels 17", "rows", "fused", "class tiles", "general", "panels 14"],
    ["general by default", "panels by default", "fused", "general odd"],
]


@pytest.fixture(scope="module")
def solo():
    import oracle as O
    out = {}
    for k, (name, (p, t, kernels)) in enumerate(KINDS.items()):
        s = E.Sectors.from_problem(p)
        s.set_tuning(**t)
        assert s.apply_kernels() == kernels, name
        psi = I.psi(4100 + k, s.dim)
        x = s.import_(torch.from_numpy(psi).to("cuda:0"))
        y = s.apply(x)
        if s.dim < 500000:
            ref = O.Sector(p.model, p.n_up, p.n_dn).apply(psi)
            assert np.linalg.norm(s.export(y).cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref), name
        out[name] = (s, x, y)
    return out


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("names", BATCHES, ids=lambda b: "-".join(n.replace(" ", "_") for n in b))
def test_batch_equals_the_problems_alone(dev, solo, names, noalloc):
    """Every output of a batch equals the problem's own application bit for
    bit, whichever left passes its problems take and in whichever order; the
    problems alone agree with the oracle (1e-12)."""
    for order in (names, names[::-1], names[1:] + names[:1]):
        S, xs, ref = zip(*(solo[n] for n in order))
        ys = [torch.full_like(x, float("nan")) for x in xs]
        E.apply_batch(list(S), list(xs), ys, noalloc=noalloc)
        for n, y, r in zip(order, ys, ref):
            assert torch.equal(y, r), (n, order)


@pytest.mark.parametrize("p,kernels", [
    (_hub(13, 4, 6), "k_hubU+k_hubD"), (_hub(11, 5, 5, ring=True), "k_hubF"), (_hub(12, 6, 5, ring=True), "k_hubU+k_hubD"),
    (_hub(13, 4, 5), "k_hubF"), (_hub(13, 5, 5, ring=True), "k_hubU+k_hubD"), (_hub(16, 8, 1), "k_hub3"),
    (_hub(17, 8, 1), "k_hub2"),
    (I.Problem(I.hubbard_chain(13, 1.0, 3.0, V=0.7), I.Cut("spatial", I.left_mask_first(6)), 5, 5), "k_spinL+k_spinR"),
    (I.Problem(I.hubbard_chain(13, 1.0, 3.0, V=0.7), I.Cut("spatial", I.left_mask_first(8)), 5, 5), "k_rows"),
    (I.Problem(I.xxz_chain(23, 1.0, 0.8), I.Cut("spatial", I.left_mask_first(16)), 11), "k_spin")],
    ids=lambda v: v if isinstance(v, str) else f"{v.model.name}_{v.n_up}_{v.n_dn}_{v.cut.left_mask}")
def test_default_tuning_at_its_limits(dev, p, kernels):
    """H psi under the default tuning on both sides of its size limits against
    the oracle (relative L2 1e-12, as every H psi test), alone and in a batch
    (bit for bit), and alpha of the first Lanczos step: <x, H x> / <x, x> to
    1e-12 of |H x| / |x|."""
    import oracle as O
    s = E.Sectors.from_problem(p)
    assert s.apply_kernels() == kernels
    psi = I.psi(4300 + s.dim % 97, s.dim)
    x = s.import_(torch.from_numpy(psi).to(dev))
    y = s.apply(x)
    ref = O.Sector(p.model, p.n_up, p.n_dn).apply(psi, use_csr=False)
    assert np.linalg.norm(s.export(y).cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref)
    z = torch.full_like(x, float("nan"))
    E.apply_batch([s], [x], [z])
    assert torch.equal(y, z)
    a, _, n2 = E.lanczos_tridiag(s, x, 1)
    assert abs(a[0] - float(x @ y) / n2) <= 1e-12 * float(y.norm()) / float(x.norm())


@pytest.mark.parametrize("name", list(KINDS))
def test_vectors_at_odd_offsets(dev, solo, name):
    """Vectors that start 8 bytes past a 16-byte boundary, alone and in a
    batch: the aligned vectors' result bit for bit."""
    s, x, y = solo[name]
    src, dst = torch.empty(s.dim + 1, dtype=x.dtype, device=dev), torch.full((s.dim + 1,), float("nan"),
                                                                             dtype=x.dtype, device=dev)
    src[1:] = x
    assert src[1:].data_ptr() % 16 == 8 and dst[1:].data_ptr() % 16 == 8
    s.apply(src[1:], out=dst[1:])
    assert torch.equal(dst[1:], y) and bool(torch.isnan(dst[0]))
    dst[1:] = float("nan")
    E.apply_batch([s], [src[1:]], [dst[1:]])
    assert torch.equal(dst[1:], y) and bool(torch.isnan(dst[0]))
