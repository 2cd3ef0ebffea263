"""GPU kernels at the edges of the ranges their launch rules switch on.

Each test runs the sizes where a rule changes the kernel, its tile or its
split (and the remainders beside them) against the CPU oracle, or against
plain torch in 64 bits on vectors the oracle's own tests already cover.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2605_07621_amd import ecut, inputs as I

pytestmark = pytest.mark.gpu


def _vec(n, seed, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    return torch.randn(n, dtype=torch.float64, device=dev, generator=g)


# chunks of the reorthogonalisation kernels: 1024 elements below 2^21, then
# 2048, 4096 and 8192 (one chunk per 1024 groups); odd lengths take the
# unaligned loads at the last pair
@pytest.mark.parametrize("n,n_up", [(10, 5), (20, 9), (24, 12), (25, 12), (26, 13)])
def test_reorth_chunk_lengths(dev, n, n_up):
    """Full reorthogonalisation over every chunk length: alpha and beta enter
    the lowest Ritz value and the Ritz vector of a fixed number of steps,
    compared with modified Gram-Schmidt (twice) in torch on the same H psi.
    Rounding of 8 orthonormalised steps stays below 1e-12 of the energy; the
    Ritz vector's is that over the gap to the next Ritz value (> 1e-2 of the
    spectrum for 8 steps), so 1e-10."""
    p = I.Problem(I.xxz_chain(n, 1.0, 0.7), I.Cut("spatial", I.left_mask_first(n // 2)), n_up)
    S = ecut.Sectors.from_problem(p)
    v0, steps = _vec(S.dim, 5 + n, dev), 8
    V, a, b = [v0 / v0.norm()], [], []
    for j in range(steps):
        w = S.apply(V[-1])
        a.append(float(w @ V[-1]))
        for _ in range(2):
            for q in V:
                w = w - (q @ w) * q
        b.append(float(w.norm()))
        V.append(w / b[-1])
    ev, U = np.linalg.eigh(np.diag(a) + np.diag(b[:-1], 1) + np.diag(b[:-1], -1))
    ref = sum(float(U[k, 0]) * V[k] for k in range(steps))
    e, _, gs = S.lanczos(v0, steps, reorth=True, fixed_steps=True, want_gs=True)
    assert abs(e - ev[0]) <= 1e-12 * abs(ev[0])
    gs = gs / gs.norm()
    gs = gs if float(gs @ ref) > 0 else -gs
    assert float((gs - ref).norm()) <= 1e-10


# the generic kernel's slices: fewer elements than one pass of a group, rows
# longer than a slice, a last slice that is empty, and problems of different
# slice counts in one batch
_SLICED = [(33, 1, 16), (34, 3, 17), (36, 4, 17), (40, 3, 20)]


def test_generic_kernel_slices_vs_oracle(dev):
    """H psi of wide rings against the oracle (relative L2 1e-12, as every
    H psi test), alone and in one batch (the same vectors bit for bit), and
    alpha of the first Lanczos step, which sums the slices' partials:
    <x, H x> / <x, x> to 1e-12 of |H x| / |x|."""
    import oracle as O
    probs = [I.Problem(I.xxz_chain(n, 1.0, 0.6, periodic=True), I.Cut("spatial", I.left_mask_first(cut)), k)
             for n, k, cut in _SLICED]
    S = [ecut.Sectors.from_problem(p) for p in probs]
    xs = [_vec(s.dim, 40 + k, dev) for k, s in enumerate(S)]
    ys = [torch.empty_like(x) for x in xs]
    ecut.apply_batch(S, xs, ys)
    for p, s, x, yb in zip(probs, S, xs, ys):
        y = s.apply(x)
        assert torch.equal(y, yb)
        ref = O.Sector(p.model, p.n_up).apply(s.export(x).cpu().numpy())
        got = s.export(y).cpu().numpy()
        assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref)
        a, _, n2 = ecut.lanczos_tridiag(s, x, 1)
        assert abs(a[0] - float(x @ y) / n2) <= 1e-12 * float(y.norm()) / float(x.norm())
