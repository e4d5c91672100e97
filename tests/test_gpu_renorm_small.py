"""dmrg_renormalize_blocks on more small blocks than run beside the others (512): these take a wavefront each
(k_renorm_small), at the edges of its tiles (4-wide k steps, 16 and 32 rows, kept states and columns), next to
blocks just above its limits and with more columns than kept states. Small integers: every product and sum is exact, and
so must be the result; the two entry points agree bit for bit on random numbers, as do the two kernels.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
lib_mod = pytest.importorskip("paper_2001_04890_amd")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DIMS = (1, 2, 4, 5, 8, 9, 15, 16, 17, 20, 31, 32, 33, 40, 70)
KEPT = {"all": lambda d: d, "within": lambda d: min(d, 32), "half": lambda d: max(1, d // 2), "one": lambda d: 1}


def run(kept, draw, copies, noalloc=False):
    kept = [kept(d) for d in DIMS]
    pairs = [(so, si) for so in range(len(DIMS)) for si in range(len(DIMS))] * copies
    Os = [draw((d, k)) for d, k in zip(DIMS, kept)]
    As = [draw((DIMS[so], DIMS[si])) for so, si in pairs]

    def offsets(sizes):
        return np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)

    o, a, r = offsets([m.size for m in Os]), offsets([m.size for m in As]), offsets([kept[so] * kept[si] for so, si in pairs])
    out = torch.full((int(r[-1]),), float("nan"), dtype=torch.float64, device="cuda:0")
    lib_mod.renormalize_blocks(DIMS, kept, o[:-1], torch.as_tensor(np.concatenate([m.ravel() for m in Os]), device="cuda:0"),
                               [p[0] for p in pairs], [p[1] for p in pairs], a[:-1],
                               torch.as_tensor(np.concatenate([m.ravel() for m in As]), device="cuda:0"), r[:-1], out,
                               noalloc=noalloc)
    got = out.cpu().numpy()
    return pairs, Os, As, [got[r[b]:r[b + 1]].reshape(kept[so], kept[si]) for b, (so, si) in enumerate(pairs)]


@pytest.mark.parametrize("kept", sorted(KEPT))
def test_many_small_blocks_are_exact(kept):
    rng = np.random.default_rng(7)
    pairs, Os, As, got = run(KEPT[kept], lambda shape: rng.integers(-3, 4, shape).astype(np.float64), 8)
    assert sum(DIMS[so] <= 32 and Os[si].shape[1] <= 32 for so, si in pairs) > 512
    for (so, si), A, m in zip(pairs, As, got):
        assert np.array_equal(m, Os[so].T @ A @ Os[si]), (DIMS[so], DIMS[si])


def test_kernels_and_entry_points_agree():
    def rand(seed):
        rng = np.random.default_rng(seed)
        return rng.normal

    many = run(KEPT["half"], lambda shape, f=rand(3): f(size=shape), 8)
    same = run(KEPT["half"], lambda shape, f=rand(3): f(size=shape), 8, noalloc=True)
    few = run(KEPT["half"], lambda shape, f=rand(3): f(size=shape), 1)
    assert all(np.array_equal(x, y) for x, y in zip(many[3], same[3]))
    assert all(np.array_equal(x, y) for x, y in zip(many[3], few[3]))   # 225 blocks: one launch, k_renorm
