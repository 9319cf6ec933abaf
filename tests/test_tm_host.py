"""Host arithmetic of the Tower Module's contractions, compiled from the library's own headers (no GPU)."""
import ctypes
import os
import subprocess

import pytest

from paper_2403_00877_amd import build as hip_build


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("tm_host")
    src, so = str(tmp / "tm_host.hip"), str(tmp / "libtm_host.so")
    with open(src, "w") as f:
        f.write('#include "dmt_tm_f32.h"\n'
                'extern "C" int first_step(int steps, int part, int log2_ks) { return f32_first_step(steps, part, log2_ks); }\n'
                'extern "C" int slice_end(int K1, int kofs, int klen) { return tm_slice_end(K1, kofs, klen); }\n'
                'static DmtPerDevice once;\n'
                'extern "C" int needed(int dev) { const bool n = once.needed(dev); once.set(dev); return n; }\n')
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + hip_build.FLAGS + ["-O0", "--cuda-host-only", "-shared", "-o", so, src],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("steps", [0, 1, 5, 64, 2 ** 27 - 1, 2 ** 27, 2 ** 27 + 3, 2 ** 28 - 16])
@pytest.mark.parametrize("log2_ks", [0, 1, 3, 4])
def test_waves_share_all_steps_of_a_float32_tile(lib, steps, log2_ks):
    """Up to the rows a weight gradient may have (B x features < 2^31, 8 to a step)."""
    parts = 1 << log2_ks
    first = [lib.first_step(steps, q, log2_ks) for q in range(parts + 1)]
    assert first == [steps * q // parts for q in range(parts + 1)]
    assert first[0] == 0 and first[-1] == steps


@pytest.mark.parametrize("K", [1, 64, 1000, 8192, 2 ** 30 + 5, 2 ** 31 - 129, 2 ** 31 - 1])
@pytest.mark.parametrize("slices", [2, 3, 16])
def test_slices_cover_all_rows_of_a_16_bit_weight_gradient(lib, K, slices):
    klen = -(-(-(-K // slices)) // 64) * 64
    at, ends = 0, []
    while at < K:
        ends.append(lib.slice_end(K, at, klen))
        assert ends[-1] == min(K, at + klen)
        at += klen
    assert ends[-1] == K and len(ends) <= slices


def test_kernel_attributes_are_set_on_every_device(lib):
    assert [lib.needed(d) for d in (0, 0, 1, 1, 0, 7, 63, 7, 63, 1)] == [1, 0, 1, 0, 0, 1, 1, 0, 0, 0]
    assert [lib.needed(d) for d in (-1, -1, 64, 64)] == [1, 1, 1, 1]        # unknown: every time
