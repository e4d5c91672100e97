"""Davidson's vector steps around the number of 1024-element chunks up to which every workgroup adds the chunk
dot products itself (128): after a few iterations from a random vector the Ritz vector is normalized, the
energy is its Rayleigh quotient and the residual norm is that of H psi - theta psi. Rounding of k <= 8
orthonormal vectors and of the projected matrix bounds the three within 1e-12, 1e-11 |theta| and 1e-10 |theta|.
"""
import pytest

from dmrg_inputs import random_vector
from helpers import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
lib_mod = pytest.importorskip("paper_2001_04890_amd")
Hop, PREC_FP64 = lib_mod.Hop, lib_mod.PREC_FP64

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("L,M,chunks", [(10, 30, (1, 128)), (14, 325, (64, 129)), (14, 360, (129, 256))])
def test_ritz_pair_is_consistent(L, M, chunks):
    hop = Hop(*synth(L, M, 1.0, 5), device=0)
    print(f"[dav chunks] L {L} M {M}: {hop.n_coeff} coefficients", flush=True)
    assert chunks[0] <= -(-hop.n_coeff // 1024) < chunks[1]
    psi = torch.as_tensor(random_vector(hop.n_coeff, 3), device=DEV)
    r = hop.davidson(psi, tol=1e-14, max_iter=8, max_sub=16)
    y = torch.empty_like(psi)
    hop.hpsi(psi, y, PREC_FP64)
    norm, theta = float(psi.norm()), float(psi @ y)
    resid = float((y - theta * psi).norm())
    print(f"[dav chunks] |psi| - 1 {norm - 1:.1e} energy {r['energy'] - theta:.1e} residual {r['resid'] - resid:.1e}", flush=True)
    assert abs(norm - 1.0) < 1e-12
    assert abs(r["energy"] - theta) < 1e-11 * max(1.0, abs(theta))
    assert abs(r["resid"] - resid) < 1e-10 * max(1.0, abs(theta))
