"""CPU check of the orders 5-7 stage on 16-element tiles (stage_bt): the kernel
source on host threads under AddressSanitizer against the FP64 oracle, in two
bf16 parts (BF16x3, bound 1e-4) and in three (FP32, bound 2e-5): every order,
ragged last tiles (K = 6, 9, 48, 51), both fluxes, right-hand side and LSRK
update."""
import numpy as np
import pytest

from test_mfma_emulation import _run, emu_exe  # noqa: F401


@pytest.mark.parametrize("n,N,flux,lsrk,split", [(1, 5, "upwind", 0, True),
                                                 (2, 5, "central", 1, True),
                                                 (1, 6, "upwind", 1, False),
                                                 (1, 7, "upwind", 1, True)])
def test_two_part_tiles(emu_exe, tmp_path, n, N, flux, lsrk, split):  # noqa: F811
    err = _run(emu_exe, tmp_path, n, N, flux, grid=5, lsrk=lsrk, split=split)
    print("per-field rel L2:", np.array2string(err, precision=2))
    assert err.max() <= 1e-4


@pytest.mark.parametrize("n,N,flux,lsrk,split", [(2, 5, "upwind", 0, True),
                                                 (1, 5, "central", 1, False),
                                                 (1, 6, "upwind", 1, True)])
def test_three_part_tiles(emu_exe, tmp_path, n, N, flux, lsrk, split):  # noqa: F811
    err = _run(emu_exe, tmp_path, n, N, flux, grid=6, lsrk=lsrk, split=split)
    print("per-field rel L2:", np.array2string(err, precision=2))
    assert err.max() <= 2e-5
