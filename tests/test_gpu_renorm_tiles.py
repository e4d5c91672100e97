"""GPU parity of the density-matrix and renormalization kernels (renorm.hip) at the edges of their tiles,
through the C-ABI, against NumPy: block sizes around 16, 32 and the 128-row chunk, kept counts around 32
and the 256-column output group, sectors that keep nothing, and psi blocks of such sizes on both sides.
Sums of n products of numbers of size 1 differ between summation orders by at most n 2^-53 times the sum of
the products' sizes; the bar is 1e-13 of the largest such sum.
"""
import numpy as np
import pytest

from dmrg_inputs import random_integrals, random_vector
from dmrg_inputs.synthetic import synthetic_block

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
lib_mod = pytest.importorskip("paper_2001_04890_amd")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("dims, kept", [
    ((1, 2, 15, 16, 17), (1, 0, 15, 3, 17)),
    ((31, 32, 33, 40), (31, 32, 33, 1)),
    ((127, 128, 129, 5), (33, 64, 65, 5)),
    ((255, 256, 257, 300), (255, 256, 257, 0)),
])
def test_renormalize_blocks_at_tile_edges(dims, kept, noalloc):
    rng = np.random.default_rng(sum(dims))
    pairs = [(i, j) for i in range(len(dims)) for j in range(len(dims))]
    O = [rng.uniform(-1, 1, (d, k)) for d, k in zip(dims, kept)]
    A = [rng.uniform(-1, 1, (dims[i], dims[j])) for i, j in pairs]
    off = lambda v: np.concatenate([[0], np.cumsum(v)]).astype(np.int64)
    o_off, a_off, r_off = off([o.size for o in O]), off([a.size for a in A]), off([kept[i] * kept[j] for i, j in pairs])
    out = torch.full((int(r_off[-1]),), np.nan, device=DEV, dtype=torch.float64)
    flat = lambda v: torch.as_tensor(np.concatenate([x.ravel() for x in v]), device=DEV)
    lib_mod.renormalize_blocks(dims, kept, o_off[:-1], flat(O), [i for i, _ in pairs], [j for _, j in pairs], a_off[:-1], flat(A),
                               r_off[:-1], out, noalloc=noalloc)
    got = out.cpu().numpy()
    for n, (i, j) in enumerate(pairs):
        ref = O[i].T @ A[n] @ O[j]
        size = np.abs(O[i]).T @ np.abs(A[n]) @ np.abs(O[j])
        g = got[r_off[n]:r_off[n + 1]].reshape(ref.shape)
        assert ref.size == 0 or np.abs(g - ref).max() <= 1e-13 * size.max(), (dims[i], dims[j])


@pytest.mark.parametrize("sizes", [(1, 3, 15, 16, 17), (31, 32, 33, 47, 49), (63, 64, 65, 97, 128)])
@pytest.mark.parametrize("side", [0, 1])
def test_density_matrices_at_tile_edges(sizes, side):
    h, eri = random_integrals(6, 3)
    ops = [("H", -1, -1)]
    left, right = (synthetic_block(s, 6, 3, 3, 2, 4096, 1.5, 7 + k, ops=ops,
                                   dim_of=lambda na, nb, k=k: sizes[(3 * na + nb + 2 * k) % len(sizes)])
                   for k, s in enumerate(("left", "right")))
    hop = lib_mod.Hop(h, eri, left, right, 3, 3, 2, device=0, share=True)
    x = random_vector(hop.n_coeff, 5)
    qn, dims, off = (hop.rdm_right_layout if side else hop.rdm_left_layout)()
    rho = torch.full((int(off[-1]),), np.nan, device=DEV, dtype=torch.float64)
    (hop.rdm_right if side else hop.rdm_left)(torch.as_tensor(x, device=DEV), rho)
    got = rho.cpu().numpy()
    # dense psi over (enlarged left, enlarged right), rows in the layouts' order
    site = [(0, 0), (1, 0), (0, 1), (1, 1)]
    def rows(blk, pairs):
        at, q = {}, {}
        for sec, st in pairs:
            k = (int(blk.qn[sec][0]) + site[st][0], int(blk.qn[sec][1]) + site[st][1])
            at[(sec, st)] = (k, q.get(k, 0))
            q[k] = q.get(k, 0) + int(blk.dim[sec])
        return at, q
    lat, lq = rows(left, [(a, s) for a in range(left.n_sec) for s in range(4)])
    rat, rq = rows(right, [(d, s) for s in range(4) for d in range(right.n_sec)])
    psi = {}
    for (a, b, c, d), (ma, md), o in zip(hop.abcd, hop.dims, hop.offsets):
        (kl, pl), (kr, pr) = lat[(a, b)], rat[(d, c)]
        m = psi.setdefault((kl, kr), np.zeros((lq[kl], rq[kr])))
        m[pl:pl + ma, pr:pr + md] = x[o:o + ma * md].reshape(ma, md)
    for i, (q, n) in enumerate(zip(qn, dims)):
        ref, size = np.zeros((n, n)), np.zeros((n, n))
        for (kl, kr), m in psi.items():
            if (kr if side else kl) == tuple(q):
                m = m.T if side else m
                ref, size = ref + m @ m.T, size + np.abs(m) @ np.abs(m).T
        assert np.abs(got[off[i]:off[i + 1]].reshape(n, n) - ref).max() <= 1e-13 * max(size.max(), 1e-300), tuple(q)
