"""dmrg_renormalize_blocks_noalloc at its limit: the longest work list that the limit allows (2^20 blocks of one
element: 56 B and one element of T each make 64 MiB) fills the device array, and one block more is refused with
nothing launched. Products of integers: exact.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
lib_mod = pytest.importorskip("paper_2001_04890_amd")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def test_longest_work_list():
    n = 1 << 20
    A = torch.arange(1, n + 2, dtype=torch.float64, device="cuda:0")
    O = torch.full((1,), 3.0, dtype=torch.float64, device="cuda:0")
    out = torch.zeros(n + 1, dtype=torch.float64, device="cuda:0")

    def call(blocks):
        at = np.arange(blocks, dtype=np.int64)
        sec = np.zeros(blocks, dtype=np.int32)
        lib_mod.renormalize_blocks([1], [1], [0], O, sec, sec, at, A, at, out, noalloc=True)

    with pytest.raises(lib_mod.DmrgError) as e:
        call(n + 1)
    assert e.value.status == -3
    assert float(out.abs().max()) == 0.0
    call(n)
    assert torch.equal(out[:n], 9.0 * A[:n]) and float(out[n]) == 0.0
