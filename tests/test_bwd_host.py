"""Host arithmetic of the sparse update, compiled from the library's own header (no GPU)."""
import ctypes
import os
import subprocess

import pytest

from paper_2403_00877_amd import build as hip_build


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("bwd_host")
    src, so = str(tmp / "bwd_host.hip"), str(tmp / "libbwd_host.so")
    with open(src, "w") as f:
        f.write('#include "dmt_bwd_plan.h"\n'
                'extern "C" int least_items(int F, int max_dim, long nnz, long* blocks, int* wide) {\n'
                '  dmt_plan p; p.F = F; p.max_dim = max_dim;\n'
                '  const BwdWs w = carve(&p, nnz, nullptr);\n'
                '  *blocks = w.nblk_sort; *wide = w.wide; return w.least_items; }\n'
                'extern "C" int items_of(unsigned len, int least) { return table_items(len, least); }\n')
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + hip_build.FLAGS + ["-O0", "--cuda-host-only", "-shared", "-o", so, src],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("F", [1, 2, 8, 26, 64, 65, 300])
@pytest.mark.parametrize("nnz", [1, 300, 16_384, 40_000, 130_000, 262_144, 500_000, 524_288, 524_289, 3_000_000])
@pytest.mark.parametrize("share", [0.0, 0.5, 0.97, 1.0])
def test_sort_blocks_of_uneven_tables(lib, F, nnz, share):
    """However the lookups are spread: no more blocks than the launch has, and no more than 64 in a table that
    blocks of 2048 records cover with 64 (a block reads the digit counts of all of its table's)."""
    blocks, wide = ctypes.c_long(), ctypes.c_int()
    for max_dim in (8, 128):
        least = lib.least_items(F, max_dim, ctypes.c_long(nnz), ctypes.byref(blocks), ctypes.byref(wide))
        assert (2 <= least <= 8) and (wide.value or least == 8)
        big = int(nnz * share)
        lens = [(nnz - big) // F] * F
        lens[F // 2] += nnz - sum(lens)
        items = [lib.items_of(n, least) for n in lens]
        per_table = [-(-n // (256 * i)) for n, i in zip(lens, items)]
        assert sum(per_table) <= blocks.value
        for n, i, nb in zip(lens, items, per_table):
            assert least <= i <= 8
            assert nb <= max(64, -(-n // 2048))
