"""The C-ABI library loads and exports every symbol include/ftkmeans.h declares (no GPU needed)."""
import ctypes
import re
from pathlib import Path

import pytest

from paper_2408_01391_amd import binding

ROOT = Path(__file__).resolve().parent.parent


def _declared():
    text = (ROOT / "include" / "ftkmeans.h").read_text()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ftk_[a-z_0-9]+)\s*\(", text)))


def test_header_and_binding_agree():
    assert _declared() == sorted(binding.EXPORTS)


def test_library_exports_every_declared_symbol():
    if not binding._LIB_PATH.exists():
        pytest.skip("libftkmeans.so not built (run python __graft_entry__.py)")
    lib = ctypes.CDLL(str(binding._LIB_PATH))
    for name in _declared():
        assert hasattr(lib, name), name
    lib.ftk_version.restype = ctypes.c_char_p
    assert b"gfx950" in lib.ftk_version()


def test_host_only_entry_points_work_without_a_gpu():
    if not binding._LIB_PATH.exists():
        pytest.skip("libftkmeans.so not built")
    from oracle import cpu as oracle
    import numpy as np
    assert np.array_equal(binding.seeded_indices(5, 1000, 50), oracle.seeded_indices(5, 1000, 50))
    assert binding.workspace_bytes(binding.F32, 1 << 20, 8, 1024) > (1 << 20) * 8
    g = binding.assign_geometry(binding.F64, 1000, 512, 64)
    assert g.lanes == 64 and g.bits == 64 and g.workgroups >= 1
    with pytest.raises(binding.FtkError):
        binding.workspace_bytes(binding.F32, 0, 8, 4)


def test_workspace_reserves_every_padded_centroid_row():
    """The prologue writes one half-norm per padded centroid row of the chosen kernel variant; the
    reservation must cover the widest padding for every K, D, dtype and fault-tolerance mode."""
    if not binding._LIB_PATH.exists():
        pytest.skip("libftkmeans.so not built")
    ks = sorted(set(list(range(1, 200, 7)) + [2 ** e + d for e in range(5, 18) for d in (-1, 0, 1, 29)]
                    + [6090, 6091, 7560, 7561, 25536, 25537, 100000, 1000003]))
    for dtype in (binding.F32, binding.F64):
        for D in (4, 8, 12, 16, 24, 32, 33, 128, 512):
            for K in ks:
                planned, reserved = binding.plan_padded_rows(dtype, max(K, 1 << 20), D, K)
                assert K <= planned <= reserved, (dtype, D, K, planned, reserved)


@pytest.mark.parametrize("dtype", [binding.F32, binding.F64])
def test_scan_reserves_every_tile_that_its_preparation_writes(dtype):
    """Two forms of the scan pad the centroids to chunks of their own (rows of 3 and 6 blocks of 16 features: 2 tiles and
    5); one launch prepares both images, for the larger of the two."""
    if not binding._LIB_PATH.exists():
        pytest.skip("libftkmeans.so not built")
    for D in list(range(17, 129, 5)) + [48, 80, 96, 128, 129, 200, 513, 1024]:
        for K in list(range(520, 8200, 32)) + [800, 1120, 2720]:
            for N in (60000, 600000):
                planned, reserved = binding.plan_padded_rows(dtype, N, D, K)
                assert planned <= reserved, (dtype, N, D, K, planned, reserved)
