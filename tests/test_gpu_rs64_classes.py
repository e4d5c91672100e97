"""The sizes of test_gpu_rs64.py (whose results are compared with the oracle there) and the set MIXED (compared
here, FP64 within 1e-12 of max|y|, as there) reach every class of the register-streamed FP64 kernel, bound on
the source's rows (k) by bound on the target's columns (q), every launch group, a group that joins the next
one's launch and one that does not. Read from the plan trace; the classes of whole task lists and of lists cut
to single tasks are counted together.
"""
import os
import re

import numpy as np
import pytest

from dmrg_inputs import random_integrals, random_vector
from dmrg_inputs.synthetic import synthetic_block
from helpers import rel_err
from oracle.hpsi import OracleHop

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
lib_mod = pytest.importorskip("paper_2001_04890_amd")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_rs64 import SIZES  # noqa: E402

TRACE = re.compile(r"\[dmrg rs64 plan\] classes([ kq:\d]*) own([ \d]+) launched([ \d]+)")


MIXED = (40, 90, 100, 45, 70, 120)     # (k, q) = (3, 4), (3, 5), (5, 2), (6, 2) among them


def problem(sizes):
    h, eri = random_integrals(6, 3)
    blocks = [synthetic_block(side, 6, 3, 3, 2, 4096, 1.5, 7 + k,
                              dim_of=lambda na, nb, k=k: sizes[(3 * na + nb + 2 * k) % len(sizes)])
              for k, side in enumerate(("left", "right"))]
    return (h, eri, *blocks, 3, 3, 2)


def build(p, cut, capfd):
    env = {"DMRG_PLAN_TRACE": "1", **({"DMRG_LDS64_ITEMS": "100000000"} if cut else {})}
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        capfd.readouterr()
        hop = lib_mod.Hop(*p, device=0)
        err = capfd.readouterr().err
    finally:
        for k, v in old.items():
            if v is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = v
    classes, own, launched = TRACE.findall(err)[-1]
    return hop, ({(int(c[1]), int(c[3])) for c in classes.split()}, [int(v) for v in own.split()],
            [int(v) for v in launched.split()])


def test_sizes_reach_every_class_and_group(capfd):
    classes, groups, joined, alone = set(), set(), set(), set()
    for sizes in (*SIZES.values(), MIXED):
        p = problem(sizes)
        for cut in (False, True):
            c, own, launched = build(p, cut, capfd)[1]
            assert sum(own) == sum(launched)
            classes |= c
            groups |= {g for g, n in enumerate(own) if n}
            joined |= {g for g, n in enumerate(own) if n and not launched[g]}
            alone |= {g for g, n in enumerate(own) if n and launched[g] == n}
    assert not {(k, q) for k in range(7) for q in range(6)} - classes
    assert groups == set(range(5))
    assert joined and alone


@pytest.mark.parametrize("cut", [False, True])
def test_mixed_sizes_match_oracle(cut, capfd):
    p = problem(MIXED)
    oh = OracleHop(*p)
    x = random_vector(oh.layout.size, 17)
    hop = build(p, cut, capfd)[0]
    xd = torch.as_tensor(x, device="cuda:0")
    yd = torch.empty_like(xd)
    hop.hpsi(xd, yd, lib_mod.PREC_FP64)
    y = yd.cpu().numpy()
    assert rel_err(y, oh.apply(x)) < 1e-12
    hop.hpsi(xd, yd, lib_mod.PREC_FP64)
    assert np.array_equal(yd.cpu().numpy(), y), "deterministic"
