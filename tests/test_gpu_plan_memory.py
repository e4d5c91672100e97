"""The padded copy of x belongs to the one-wavefront kernel: a plan whose tasks all run in the other FP64 kernels
has none, and its H.psi is that of a plan with the copy (single-tile sources in the one-wavefront kernel) within
1e-13 of max|y| (summation order only). Read from the plan trace, which names the copy's size.
"""
import os
import re

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


def test_no_operand_pool_without_its_kernels(capfd):
    """With the register-streamed kernel off and no sector above 96 nothing reads the FP64 operand pool: the handle's
    device data is less than with it."""
    p = synth(12, 150, 0.8, 5)
    data = []
    for env in ({}, {"DMRG_LDS64": "0"}):
        old = os.environ.get("DMRG_LDS64")
        os.environ.update(env, DMRG_BUILD_TRACE="1")
        try:
            capfd.readouterr()
            hop = lib_mod.Hop(*p, device=0)
            err = capfd.readouterr().err
        finally:
            os.environ.pop("DMRG_BUILD_TRACE")
            if env:
                os.environ.pop("DMRG_LDS64")
                if old is not None:
                    os.environ["DMRG_LDS64"] = old
        assert int(hop.dims.max()) <= 96
        data.append(float(re.findall(r"device memory: ([\d.]+) MB data", err)[-1]))
    print(f"[plan memory] {data}", flush=True)
    assert data[1] < data[0]
