"""GPU parity of the register-streamed FP64 H.psi kernel (hpsi_rs64.hip) against the FP64 oracle at the
edges of its tiles, through the C-ABI: sector sizes around every 4-wide k step, 16-wide tile and
class bound up to its 128 rows and columns, one size beyond it (whose tasks go to the large-block
paths), with the default plan and with task lists cut to the floor of the item cost (many partial
tiles). Bar: FP64 within 1e-12 of max|y| (summation order only), deterministic bit for bit.
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
    "1..5": (1, 2, 3, 4, 5),
    "16": (15, 16, 17, 8, 9, 12, 13),
    "32..49": (31, 32, 33, 47, 48, 49, 1),
    "64..97": (63, 64, 65, 96, 97, 20, 5),
    "112..128": (112, 113, 127, 128, 100, 3),
    "128..130": (128, 129, 130, 7, 40),
}


@pytest.fixture(scope="module")
def problems():
    made = {}

    def get(name):
        if name not in made:
            sizes = SIZES[name]
            h, eri = random_integrals(6, 3)
            blocks = [synthetic_block(side, 6, 3, 3, 2, 4096, 1.5, 7 + k,
                                      dim_of=lambda na, nb, k=k: sizes[(3 * na + nb + 2 * k) % len(sizes)])
                      for k, side in enumerate(("left", "right"))]
            p = (h, eri, *blocks, 3, 3, 2)
            oh = OracleHop(*p)
            x = random_vector(oh.layout.size, 17)
            made[name] = (p, x, oh.apply(x))
        return made[name]

    return get


@pytest.mark.parametrize("cut", [False, True])
@pytest.mark.parametrize("sizes", list(SIZES))
def test_rs64_matches_oracle(problems, sizes, cut):
    p, x, ref = problems(sizes)
    old = os.environ.get("DMRG_LDS64_ITEMS")
    if cut:
        os.environ["DMRG_LDS64_ITEMS"] = "100000000"
    try:
        hop = Hop(*p, device=0)
    finally:
        if cut:
            os.environ.pop("DMRG_LDS64_ITEMS")
            if old is not None:
                os.environ["DMRG_LDS64_ITEMS"] = old
    xd = torch.as_tensor(x, device=DEV)
    yd = torch.empty_like(xd)
    hop.hpsi(xd, yd, PREC_FP64)
    y = yd.cpu().numpy()
    print(f"[rs64] {sizes} cut {cut}: rel err {rel_err(y, ref):.2e}", flush=True)
    assert rel_err(y, ref) < FP64_TOL
    hop.hpsi(xd, yd, PREC_FP64)
    assert np.array_equal(yd.cpu().numpy(), y), "deterministic"
