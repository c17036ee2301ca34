"""CPU test of the limit on a batch's wide maps: a partition's cursor, which an overflowing map may run
past its region by as many records as the map has, stays within the 32 bits that runs are placed by."""
import ctypes

from paper_2508_11443_amd import fks


def test_cursors_stay_in_32_bits():
    import torch  # noqa: F401  (its HIP runtime first: the library shares it)
    lib = fks.library()
    most = getattr(lib, "_ZN3fks14wide_parts_maxEv")
    most.argtypes, most.restype = [], ctypes.c_uint64
    scratch = getattr(lib, "_ZN3fks18wide_scratch_bytesEjmm")
    scratch.argtypes, scratch.restype = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint64], ctypes.c_size_t
    # a partition's share of the scratch: 12 bytes for each record of its region, two words and a list entry
    parts = 1 << 16
    region = ((scratch(1, 2 * parts, 1) - scratch(1, parts, 1)) // parts - 20) // 12
    assert region % 256 == 0 and 1024 < region < 4096
    assert most() * region + 65536 <= 1 << 32
    assert most() >= 2_700_000
