"""Slot tables of the Hubbard up/down kernels against the hopping operators.

The fused and the two-pass kernels read the down-spin hops from slots (one per
site pair) and the up-spin hops from CSR rows, and scale both by one number
where every hop has the same value.  Here the operator that they apply is
rebuilt from those host tables, through a small C++ reader of the handle, and
compared with the sum over the listed bonds.  CPU only, but for the parity
test at the end.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2605_07621_amd import ecut as E, inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

READER = r"""
#include "ecut_internal.h"
extern "C" int slot_tables(const ecut_sectors *s, int *uniform, int *n_slots, double *hop, int *col, double *val) {
    if (!s->hub6_ok) return 1;
    *uniform = s->h6_uniform;
    *n_slots = s->h6_maxq;
    *hop = s->h6_hop;
    const size_t n = (size_t)s->h6_maxq * s->blocks[0].d_r;
    if (col)
        for (size_t k = 0; k < n; ++k) {
            col[k] = s->h6_col[k];
            val[k] = s->h6_uniform ? s->h6_hop : s->h6_val[k];
        }
    return 0;
}
extern "C" void up_rows(const ecut_sectors *s, int *ptr, int *col, double *val) {
    const int n = s->blocks[0].d_l;
    for (int a = 0; a <= n; ++a) ptr[a] = s->hl_ptr[a];
    for (int k = 0; col && k < ptr[n]; ++k) {
        col[k] = s->hl_col[k];
        val[k] = s->h6_uniform ? s->h6_hop : s->hl_val[k];
    }
}
extern "C" void down_words(const ecut_sectors *s, unsigned *w) {
    for (int c = 0; c < s->blocks[0].d_r; ++c) w[c] = s->hub_rw32[c];
}
"""


@pytest.fixture(scope="module")
def reader(tmp_path_factory):
    d = tmp_path_factory.mktemp("reader")
    src, lib = d / "reader.cpp", d / "libreader.so"
    src.write_text(READER)
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-w",
                        "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "paper_2605_07621_amd", "csrc"), str(src),
                        "-o", str(lib)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return ctypes.CDLL(str(lib))


def _hops(words, pairs, t):
    """Dense sum over the listed bonds of -t_b (c+_i c_j + h.c.) on the words."""
    index = {int(w): k for k, w in enumerate(words)}
    H = np.zeros((len(words), len(words)))
    for (i, j), tb in zip(pairs, t):
        lo, hi = min(i, j), max(i, j)
        between = ((1 << hi) - 1) & ~((1 << (lo + 1)) - 1)
        for w, k in index.items():
            if ((w >> i) & 1) != ((w >> j) & 1):
                H[k, index[w ^ (1 << i) ^ (1 << j)]] -= tb * (-1) ** bin(w & between).count("1")
    return H


def _model(n, pairs, t):
    return I.Model("hubbard", n, np.asarray(pairs, dtype=np.int32).reshape(-1, 2), t=np.asarray(t, dtype=float),
                   u=np.full(n, 3.0), name="pairs")


CHAIN6 = [(i, i + 1) for i in range(5)]
# (name, model, n_up, n_dn): pairs listed once, in both directions, as the two
# bonds of a short ring, as a 2x2 torus, in mixed numbers whose sums agree or
# do not, and with sums of zero
MODELS = [
    ("chain", _model(6, CHAIN6, [1.0] * 5), 3, 3),
    ("both directions", _model(6, CHAIN6 + [(j, i) for i, j in CHAIN6], [0.5] * 10), 3, 3),
    ("both directions, one spin full", _model(6, CHAIN6 + [(j, i) for i, j in CHAIN6], [0.5] * 10), 6, 3),
    ("two-site ring", _model(2, [(0, 1), (1, 0)], [1.0, 1.0]), 1, 1),
    ("2x2 torus", _model(4, [(0, 1), (1, 0), (2, 3), (3, 2), (0, 2), (2, 0), (1, 3), (3, 1)], [1.0] * 8), 1, 1),
    ("2x2 torus, half filling", _model(4, [(0, 1), (1, 0), (2, 3), (3, 2), (0, 2), (2, 0), (1, 3), (3, 1)], [1.0] * 8),
     2, 2),
    ("mixed numbers, one sum", _model(5, [(0, 1), (1, 0), (1, 2), (3, 2), (2, 3), (3, 2), (3, 4)],
                                      [0.25, 0.75, 1.0, 0.5, 0.25, 0.25, 1.0]), 2, 3),
    ("mixed numbers, one value", _model(5, [(0, 1), (1, 0), (1, 2), (3, 2), (3, 4)], [1.0] * 5), 2, 3),
    ("a pair that cancels", _model(5, CHAIN6[:4] + [(0, 1), (1, 0)], [1.0, 1.0, 1.0, 1.0, -0.5, -0.5]), 3, 2),
    ("every pair cancels", _model(4, [(0, 1), (1, 0), (2, 3), (2, 3)], [1.0, -1.0, 0.5, -0.5]), 2, 1),
    ("ring, each bond three times", _model(5, [(i, (i + 1) % 5) for i in range(5)] * 3, [0.25] * 5 + [0.5] * 5 + [0.25] * 5),
     2, 2),
]


@pytest.mark.parametrize("name,model,n_up,n_dn", MODELS, ids=[m[0] for m in MODELS])
def test_slot_operator_is_the_sum_over_bonds(reader, name, model, n_up, n_dn):
    """Down-spin slots and up-spin rows, scaled as the kernels scale them,
    equal the dense sum over the listed bonds (all numbers are multiples of
    1/4: exact)."""
    S = E.Sectors.from_problem(I.Problem(model, I.Cut("updn"), n_up, n_dn), host_only=True)
    dl, dr = int(S.blocks()[0][2]), int(S.blocks()[0][3])
    u, ns, hop = ctypes.c_int(), ctypes.c_int(), ctypes.c_double()
    h = S.h
    assert reader.slot_tables(h, ctypes.byref(u), ctypes.byref(ns), ctypes.byref(hop), None, None) == 0
    col, val = np.zeros((ns.value, dr), np.int32), np.zeros((ns.value, dr))
    reader.slot_tables(h, ctypes.byref(u), ctypes.byref(ns), ctypes.byref(hop), ctypes.c_void_p(col.ctypes.data),
                       ctypes.c_void_p(val.ctypes.data))
    w = np.zeros(dr, np.uint32)
    reader.down_words(h, ctypes.c_void_p(w.ctypes.data))
    dn = np.zeros((dr, dr))
    for k in range(ns.value):
        for c in range(dr):
            if col[k, c] >= 0:
                dn[c, col[k, c]] += val[k, c]
    assert np.array_equal(dn, _hops(w, model.bonds, model.t))
    ptr = np.zeros(dl + 1, np.int32)
    reader.up_rows(h, ctypes.c_void_p(ptr.ctypes.data), None, None)
    ucol, uval = np.zeros(ptr[-1] + 1, np.int32), np.zeros(ptr[-1] + 1)
    reader.up_rows(h, ctypes.c_void_p(ptr.ctypes.data), ctypes.c_void_p(ucol.ctypes.data), ctypes.c_void_p(uval.ctypes.data))
    up = np.zeros((dl, dl))
    for a in range(dl):
        for k in range(ptr[a], ptr[a + 1]):
            up[a, ucol[k]] += uval[k]
    assert np.array_equal(up, _hops(S.words(0)[0], model.bonds, model.t))


def _gpu_problems():
    out = [I.Problem(m, I.Cut("updn"), a, b) for _, m, a, b in MODELS]
    chain = [(i, i + 1) for i in range(11)]
    both = _model(12, chain + [(j, i) for i, j in chain], [0.5] * 22)
    out.append(I.Problem(both, I.Cut("updn"), 6, 6))        # one value: fused kernel at 853,776 amplitudes
    ring = [(i, (i + 1) % 12) for i in range(12)]
    out.append(I.Problem(_model(12, ring * 2, [0.5] * 24), I.Cut("updn"), 6, 6))   # signed: two passes
    out.append(I.Problem(_model(6, CHAIN6 + [(1, 0)], [1.0] * 6), I.Cut("updn"), 6, 3))   # class tiles, a low pair twice
    for cut, q in ((0b111, (3, 3)), (0b1011, (2, 4))):      # the spatial cut and a spin cut of the same pairs
        m = _model(6, CHAIN6 + [(j, i) for i, j in CHAIN6] + [(0, 5), (5, 0)], [0.5] * 12)
        out.append(I.Problem(I.Model(**dict(m.__dict__, v=np.full(12, 0.25))), I.Cut("spatial", cut), *q))
        out.append(I.Problem(I.Model("spin", 6, m.bonds, jxy=np.full(12, 0.5), jz=np.full(12, 0.75), name="pairs"),
                             I.Cut("spatial", cut), 3))
    return out


@pytest.mark.gpu
def test_repeated_pairs_vs_oracle(dev):
    """H psi of these models by the default tuning, by every variant the
    handle takes and in one batch (the default's vectors bit for bit) against
    the oracle (relative L2 1e-12, as every H psi test)."""
    torch = pytest.importorskip("torch")
    import oracle as O
    S, xs, ys = [], [], []
    for k, p in enumerate(_gpu_problems()):
        s = E.Sectors.from_problem(p)
        psi = I.psi(3100 + k, s.dim)
        x = s.import_(torch.from_numpy(psi).to(dev))
        ref = O.Sector(p.model, p.n_up, p.n_dn).apply(psi)
        for v in (None, 0, 1, 2, 3, 4, 5, 6, 7):
            try:
                s.set_tuning(**({} if v is None else dict(variant=v, n_xcd=8)))
            except E.EcutError:
                continue
            y = s.apply(x)
            got = s.export(y).cpu().numpy()
            assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref), (k, p.model.name, v)
            if v is None:
                ys.append(y)
        s.set_tuning()
        S.append(s), xs.append(x)
    out = [torch.full_like(x, float("nan")) for x in xs]
    E.apply_batch(S, xs, out)
    for a, b in zip(ys, out):
        assert torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("n,a,b", [(7, 5, 6), (8, 4, 1), (10, 2, 8), (11, 5, 5), (12, 3, 6)])
def test_one_u_with_uneven_hops_vs_oracle(dev, n, a, b):
    """One U on every site and hops of several values, by every variant: the
    whole-row kernel of uneven models keeps a table of U by byte of the word
    even where one U would do (relative L2 1e-12)."""
    torch = pytest.importorskip("torch")
    import oracle as O
    t = np.random.default_rng(n).normal(size=n)
    p = I.Problem(_model(n, [(i, (i + 1) % n) for i in range(n)], t), I.Cut("updn"), a, b)
    s = E.Sectors.from_problem(p)
    psi = I.psi(3300 + n, s.dim)
    x = s.import_(torch.from_numpy(psi).to(dev))
    ref = O.Sector(p.model, a, b).apply(psi)
    for v in (0, 1, 2, 4, 6):
        for kw in (dict(n_xcd=8), dict(n_xcd=1, grid=4, row_order=1)):
            try:
                s.set_tuning(variant=v, **kw)
            except E.EcutError:
                continue
            got = s.export(s.apply(x)).cpu().numpy()
            assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref), (v, kw)
