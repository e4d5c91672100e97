"""GPU parity of the FP64 two-pass path (hpsi_big64.hip) against the FP64 oracle at the edges of its work:
extents around whole 4-row groups and 16-row tiles, around the tile counts where a block is cut into one
more part (4, 8, 9, 12 tiles), odd numbers of 4-wide k steps, tiny targets with large sources and large
targets with tiny ones, with the default plan and with task ranges of 4 tiles (partial sums). Every target
takes the path: the sectors within 128 x 128 have larger sources. Bar: 1e-12 of max|y| (summation order
only), deterministic bit for bit.
"""
import os

import numpy as np
import pytest

from dmrg_inputs import random_integrals, random_vector
from dmrg_inputs.synthetic import synthetic_block
from oracle.hpsi import OracleHop
from helpers import rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
lib_mod = pytest.importorskip("paper_2001_04890_amd")
Hop, PREC_FP64 = lib_mod.Hop, lib_mod.PREC_FP64

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = torch.device("cuda:0")
FP64_TOL = 1e-12
SIZES = {
    "129..145": (129, 131, 133, 144, 145),
    "tiny and large": (1, 200, 3, 17, 193, 5),
    "tile counts": (64, 65, 128, 129, 192, 193),
    "k steps": (4, 133, 140, 12, 148, 8),
}


@pytest.mark.parametrize("cut", [False, True])
@pytest.mark.parametrize("sizes", list(SIZES))
def test_big64_matches_oracle(sizes, cut):
    dims = SIZES[sizes]
    h, eri = random_integrals(6, 3)
    blocks = [synthetic_block(side, 6, 3, 3, 2, 4096, 1.5, 7 + k,
                              dim_of=lambda na, nb, k=k: dims[(3 * na + nb + 2 * k) % len(dims)])
              for k, side in enumerate(("left", "right"))]
    p = (h, eri, *blocks, 3, 3, 2)
    oh = OracleHop(*p)
    x = random_vector(oh.layout.size, 17)
    ref = oh.apply(x)
    env = {"DMRG_BIG_STAGES": "4", "DMRG_BIG_TBUDGET_MB": "16"} if cut else {}
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        hop = Hop(*p, device=0)
    finally:
        for k, v in old.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v
    xd = torch.as_tensor(x, device=DEV)
    yd = torch.empty_like(xd)
    hop.hpsi(xd, yd, PREC_FP64)
    y = yd.cpu().numpy()
    print(f"[big64] {sizes} cut {cut}: rel err {rel_err(y, ref):.2e}", flush=True)
    assert rel_err(y, ref) < FP64_TOL
    hop.hpsi(xd, yd, PREC_FP64)
    assert np.array_equal(yd.cpu().numpy(), y), "deterministic"
