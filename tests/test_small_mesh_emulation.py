"""CPU check of the one-element-per-workgroup stage at orders 2-4 (contexts of
few 16-element tiles): the kernel source on host threads under AddressSanitizer
against the FP64 oracle, BF16x3 (1e-4), FP32 (2e-5) and FP64 (1e-12)."""
import numpy as np
import pytest

from test_mfma_emulation import _run, emu_exe  # noqa: F401


@pytest.mark.parametrize("n,N,grid,flux,lsrk,split,bound",
                         [(1, 2, 8, "upwind", 1, True, 1e-4), (1, 3, 8, "central", 0, False, 1e-4),
                          (1, 4, 8, "upwind", 0, True, 1e-4), (1, 2, 9, "central", 0, True, 2e-5),
                          (1, 3, 9, "upwind", 1, True, 2e-5), (1, 4, 9, "upwind", 0, False, 2e-5),
                          (1, 2, 10, "upwind", 0, False, 1e-12),
                          (1, 3, 10, "upwind", 1, True, 1e-12),
                          (1, 4, 10, "central", 0, True, 1e-12)])
def test_one_element_kernel_at_low_orders(emu_exe, tmp_path, n, N, grid, flux, lsrk,  # noqa: F811
                                          split, bound):
    err = _run(emu_exe, tmp_path, n, N, flux, grid=grid, lsrk=lsrk, split=split)
    print("per-field rel L2:", np.array2string(err, precision=2))
    assert err.max() <= bound
