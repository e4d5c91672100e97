"""GPU parity of the split-precision H.psi kernels (hpsi_lds.hip row mode and task mode, hpsi_big.hip) against
the FP64 oracle at the edges of their tiles: sizes around 16-row tiles, 32-wide k tiles, two row tiles per
wavefront, the 64 and 96 bounds of the row-mode classes, one size above them and the extents where a large
block is cut into one more part, with the default plan and with task lists cut to the floor of the item cost.
Bar: the error bound of the 2-term BF16 split, element by element (helpers.assert_split_bound);
deterministic bit for bit.
"""
import os

import numpy as np
import pytest

from dmrg_inputs import random_integrals, random_vector
from dmrg_inputs.synthetic import synthetic_block
from oracle.hpsi import OracleHop
from helpers import assert_split_bound

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
lib_mod = pytest.importorskip("paper_2001_04890_amd")
Hop, PREC_SPLIT2 = lib_mod.Hop, lib_mod.PREC_SPLIT2

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = torch.device("cuda:0")
SIZES = {
    "1..33": (1, 15, 16, 17, 31, 32, 33),
    "32..65": (47, 48, 49, 63, 64, 65, 5),
    "80..97": (80, 81, 95, 96, 97, 12),
    "parts": (64, 65, 128, 129, 192, 3),
}


@pytest.mark.parametrize("cut", [False, True])
@pytest.mark.parametrize("sizes", list(SIZES))
def test_split_matches_oracle(sizes, cut):
    dims = SIZES[sizes]
    h, eri = random_integrals(6, 3)
    blocks = [synthetic_block(side, 6, 3, 3, 2, 4096, 1.5, 7 + k,
                              dim_of=lambda na, nb, k=k: dims[(3 * na + nb + 2 * k) % len(dims)])
              for k, side in enumerate(("left", "right"))]
    p = (h, eri, *blocks, 3, 3, 2)
    oh = OracleHop(*p)
    x = random_vector(oh.layout.size, 17)
    env = {"DMRG_LDS_ITEMS": "100000000", "DMRG_BIG_STAGES": "4", "DMRG_BIG_TBUDGET_MB": "16"} if cut else {}
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        hop = Hop(*p, device=0, want_split=True)
    finally:
        for k, v in old.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v
    xd = torch.as_tensor(x, device=DEV)
    yd = torch.empty_like(xd)
    hop.hpsi(xd, yd, PREC_SPLIT2)
    y = yd.cpu().numpy()
    assert_split_bound(y, oh.apply(x), oh.magnitude(x), f"{sizes} cut {cut}")
    hop.hpsi(xd, yd, PREC_SPLIT2)
    assert np.array_equal(yd.cpu().numpy(), y), "deterministic"
