"""The padded copy of x belongs to the one-wavefront kernel: a plan whose tasks all run in the other FP64 kernels
has none, and its H.psi is that of a plan with the copy (single-tile sources in the one-wavefront kernel) within
1e-13 of max|y| (summation order only). Read from the plan trace, which names the copy's size.
"""
import os

import pytest

from dmrg_inputs import random_vector
from helpers import rel_err, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
lib_mod = pytest.importorskip("paper_2001_04890_amd")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def run(p, env, capfd):
    env = dict(env, DMRG_PLAN_TRACE="1")
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
    x = torch.as_tensor(random_vector(hop.n_coeff, 3), device="cuda:0")
    y = torch.empty_like(x)
    hop.hpsi(x, y, lib_mod.PREC_FP64)
    return y.cpu().numpy(), "[dmrg plan]" in err


@pytest.mark.parametrize("L,M", [(8, 20), (12, 150)])
def test_no_padded_copy_without_one_wavefront_tasks(L, M, capfd):
    p = synth(L, M, 0.8, 5)
    y, copy = run(p, {}, capfd)
    y1, copy1 = run(p, {"DMRG_LDS64_SMALL": "0"}, capfd)
    assert not copy and copy1
    assert rel_err(y, y1) < 1e-13
