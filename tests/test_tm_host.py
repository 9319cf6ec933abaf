"""Host arithmetic of the Tower Module's contractions, compiled from the library's own headers (no GPU)."""
import ctypes
import os
import subprocess

import pytest
import torch

import paper_2403_00877_amd as dmt
from paper_2403_00877_amd import build as hip_build


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("tm_host")
    src, so = str(tmp / "tm_host.hip"), str(tmp / "libtm_host.so")
    with open(src, "w") as f:
        # (the two runtime calls of dmt_allow_lds, so that it can be watched on devices that are not there)
        f.write('#include <hip/hip_runtime.h>\n'
                'static int g_dev, g_sets, g_fail;\n'
                'static hipError_t fake_get(int* d) { *d = g_dev; return hipSuccess; }\n'
                'static hipError_t fake_set(const void*, hipFuncAttribute, int) { ++g_sets; return g_fail ? hipErrorInvalidValue : hipSuccess; }\n'
                '#define hipGetDevice fake_get\n'
                '#define hipFuncSetAttribute fake_set\n'
                '#include "dmt_tm_f32.h"\n'
                'static DmtPerDevice lds;\n'
                'extern "C" int allow_lds(int dev, int fail) { g_dev = dev; g_fail = fail; g_sets = 0; dmt_allow_lds(lds, &lds, 1); return g_sets; }\n'
                'extern "C" int first_step(int steps, int part, int log2_ks) { return f32_first_step(steps, part, log2_ks); }\n'
                'extern "C" int share_begin(int steps, int part, int log2_ks, int batches) { return f32_share_begin(steps, part, log2_ks, batches); }\n'
                '// n[i] groups of M[i] x N[i], K[i]; each arranged group: which kind it is and the log2 of its waves a tile\n'
                'extern "C" int arrange(int kinds, const int* n, const int* M, const int* N, const int* K, int epi, int forward, int* kind, int* log2_ks) {\n'
                '  std::vector<TmF32Group> v;\n'
                '  for (int i = 0; i < kinds; ++i) for (int j = 0; j < n[i]; ++j) { TmF32Group g{}; g.M = M[i]; g.N = N[i]; g.K1 = K[i]; g.epi = epi; g.lda1 = i; v.push_back(g); }\n'
                '  f32_arrange(v, forward != 0);\n'
                '  for (size_t i = 0; i < v.size(); ++i) { kind[i] = v[i].lda1; log2_ks[i] = v[i].log2_ks; }\n'
                '  return (int)v.size(); }\n'
                '// T like dot towers of nf features of n columns to O outputs, beside one of a kind and nf2 features (or -1)\n'
                'extern "C" int one_kernel(int T, int nf, int n, int O, long B, int fuse, int kind, int nf2) {\n'
                '  dmt_plan p; p.sw.tm_fuse = fuse; p.T = T; p.tower_ntab.assign(T, nf); p.tower_uniform_dim.assign(T, n);\n'
                '  dmt_tm_params q{}; q.kind = DMT_TM_DOT_LINEAR; q.out_dim = O;\n'
                '  std::vector<dmt_tm_params> tp(T, q);\n'
                '  if (kind >= 0) { q.kind = kind; tp.push_back(q); ++p.T; p.tower_ntab.push_back(nf2); p.tower_uniform_dim.push_back(n); }\n'
                '  return dot_one_kernel(&p, 0, O, dot_dgrad_of(&p, tp.data(), B)); }\n'
                'extern "C" int slice_end(int K1, int kofs, int klen) { return tm_slice_end(K1, kofs, klen); }\n'
                '// blocks of a launch of n like groups; *tiles its tiles\n'
                'extern "C" long blocks_of(int n, int M, int N, int K0, int K1, int reps, long* tiles) {\n'
                '  dmt_plan p; TmLaunch L; L.ngroups = n; bool big;\n'
                '  for (int i = 0; i < n; ++i) { TmGroup g{}; g.M = M; g.N = N; g.K0 = K0; g.K1 = K1; g.reps = reps; L.g[i] = g; }\n'
                '  const long b = tile_launch(&p, L, false, KIND_PLAIN, &big);\n'
                '  *tiles = 0; for (int i = 0; i < n; ++i) *tiles += tiles_of(L.g[i], big ? 256 : 128);\n'
                '  return big ? b : -b; }\n'
                'extern "C" int forward_tile(int n, int M, int N, int K1, int dK, int epi, int dots) {\n'
                '  dmt_plan p; TmGroup g[kMaxGroups] = {};\n'
                '  for (int i = 0; i < n; ++i) { g[i].M = M; g[i].N = N; g[i].K1 = K1 + i * dK; g[i].epi = epi; }\n'
                '  return take_small(&p, g, n, dots != 0) ? 32 : take_big(&p, g, n) ? 256 : 128; }\n'
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


@pytest.mark.parametrize("steps", [0, 1, 3, 4, 5, 48, 63, 2 ** 27 + 3, 2 ** 28 - 15])
@pytest.mark.parametrize("log2_ks", [0, 2, 4])
def test_waves_shares_are_whole_batches(lib, steps, log2_ks):
    begin = [lib.share_begin(steps, q, log2_ks, 1) for q in range((1 << log2_ks) + 1)]
    assert begin[0] == 0 and begin[-1] == steps and begin == sorted(begin)
    assert all(b % 4 == 0 or b == steps for b in begin)


@pytest.mark.parametrize("steps", [0, 1, 14, 81, 2 ** 28 - 15])
@pytest.mark.parametrize("log2_ks", [0, 1, 4])
def test_waves_shares_of_a_backward_are_as_even_as_steps_allow(lib, steps, log2_ks):
    begin = [lib.share_begin(steps, q, log2_ks, 0) for q in range((1 << log2_ks) + 1)]
    shares = [b - a for a, b in zip(begin, begin[1:])]
    assert begin[0] == 0 and begin[-1] == steps and max(shares) - min(shares) <= 1


def arrange(lib, kinds, epi=0, forward=True):
    """kinds: (groups, M, N, K); (kind, log2 of the waves a tile) of every group in order."""
    cols = [(ctypes.c_int * len(kinds))(*c) for c in zip(*kinds)]
    total = sum(k[0] for k in kinds)
    kind, log2_ks = (ctypes.c_int * total)(), (ctypes.c_int * total)()
    assert lib.arrange(len(kinds), *cols, epi, int(forward), kind, log2_ks) == total
    return list(zip(kind, log2_ks))


@pytest.mark.parametrize("kinds,epi,forward,want", [
    # the towers beyond a launch of 16 do not take waves from it: 2048 tiles of 24 steps there, 512 in the next
    ([(20, 2048, 64, 192)], 0, True, [1] * 16 + [2] * 4),
    ([(26, 2048, 64, 64)], 3, False, [1] * 26),
    # 16 cross layers of 376 tiles are a round and a half: three rounds of half as long; the other four fit one
    ([(20, 6000, 64, 64)], 2, True, [1] * 20),
    # short of a second round that would be half empty
    ([(2, 6000, 64, 286)], 0, True, [2] * 2),
    # data gradients of 8 steps beside weight gradients of 256
    ([(4, 2048, 416, 64), (4, 64, 416, 2048)], 3, False, [4] * 4 + [0] * 4),
    # a wave may keep 32 steps in a second round
    ([(1, 512, 2560, 512), (1, 512, 2560, 512)], 3, False, [1] * 2),
    ([(1, 32, 32, 8), (1, 33, 1, 24)], 0, True, [0, 0]),
    # (data gradients of 4 steps are as long as the weight gradients' halves of 8)
    ([(2, 64, 64, 32), (2, 32, 64, 64)], 3, False, [1, 1, 0, 0]),
])
def test_waves_of_float32_tiles_are_counted_by_the_launch(lib, kinds, epi, forward, want):
    assert [l for _, l in arrange(lib, kinds, epi, forward)] == want


@pytest.mark.parametrize("forward", [True, False])
def test_float32_launches_start_with_the_longest_waves(lib, forward):
    kinds = [(3, 900, 50, 1391), (14, 107, 64, 96), (9, 640, 32, 107), (4, 32, 64, 40000)]
    got = arrange(lib, kinds, 3, forward)
    assert sorted(k for k, _ in got) == sorted(i for i, k in enumerate(kinds) for _ in range(k[0]))
    for first in range(0, len(got), 16):
        waves = [(kinds[k][3] + 7) // 8 >> l for k, l in got[first:first + 16]]
        assert waves == sorted(waves, reverse=True)
        assert all(l == 0 or (kinds[k][3] + 7) // 8 >> l >= 4 for k, l in got[first:first + 16])


def one_kernel(lib, T, nf, n, O, B, fuse=1, beside=(-1, 0)):
    return lib.one_kernel(T, nf, n, O, ctypes.c_long(B), fuse, *beside)


@pytest.mark.parametrize("T,nf,n,O,B,want", [
    (8, 8, 128, 256, 8192, 1), (4, 7, 128, 256, 2003, 1), (4, 4, 64, 256, 200, 1), (1, 8, 32, 128, 1, 1),
    # few blocks and many outputs: the contractions' more tiles are faster
    (4, 8, 32, 512, 300, 0), (4, 8, 128, 2048, 300, 0), (4, 6, 32, 2048, 2000, 0), (1, 2, 32, 640, 1, 1), (1, 2, 32, 641, 1, 0),
    (1, 8, 32, 384, 4096, 1), (1, 8, 32, 385, 4096, 0), (4, 8, 64, 1024, 4096, 1), (8, 8, 128, 2048, 512, 0),
    (9, 8, 128, 2048, 512, 1),           # beside their dot terms, more than one launch of contractions
    (4, 9, 32, 64, 4096, 0), (4, 8, 40, 64, 4096, 0), (4, 1, 32, 64, 4096, 0),
])
def test_when_a_dot_towers_data_gradient_is_one_kernel(lib, T, nf, n, O, B, want):
    assert one_kernel(lib, T, nf, n, O, B) == want
    assert one_kernel(lib, T, nf, n, O, B, fuse=0) == 0
    assert one_kernel(lib, T, nf, n, O, B, fuse=2) == (2 <= nf <= 8 and n % 32 == 0)


@pytest.mark.parametrize("B,linear,dots", [(1000, 0, 0), (2047, 0, 0), (2048, 1, 0), (3906, 1, 0), (3907, 1, 1)])
def test_a_dot_towers_data_gradient_beside_other_towers(lib, B, linear, dots):
    """8 features of 128 columns: in a launch of its own where it saves more than that."""
    assert one_kernel(lib, 1, 8, 128, 256, B) == 1
    for kind in (dmt.binding.DMT_TM_LINEAR, dmt.binding.DMT_TM_LINEAR_RELU, dmt.binding.DMT_TM_DLRM):
        assert one_kernel(lib, 1, 8, 128, 256, B, beside=(kind, 8)) == linear
    assert one_kernel(lib, 1, 8, 128, 256, B, beside=(dmt.binding.DMT_TM_DOT_LINEAR, 9)) == dots
    assert one_kernel(lib, 1, 8, 128, 256, B, beside=(dmt.binding.DMT_TM_DOT_LINEAR, 2)) == 1
    assert one_kernel(lib, 1, 8, 128, 256, B, beside=(dmt.binding.DMT_TM_CROSS_LINEAR, 8)) == 1
    assert one_kernel(lib, 1, 8, 128, 256, B, 2, (dmt.binding.DMT_TM_DOT_LINEAR, 9)) == 1
    assert one_kernel(lib, 9, 8, 128, 256, B, 1, (dmt.binding.DMT_TM_DOT_LINEAR, 9)) == 1


@pytest.mark.parametrize("T,nf,n,O,B,copy", [
    (4, 7, 128, 256, 2003, 0), (4, 8, 128, 2048, 300, 0),      # one kernel, with a layout of its own; an even number of terms
    (4, 7, 128, 2048, 300, 1), (4, 10, 32, 64, 300, 1), (2, 3, 24, 40, 70, 1),
])
def test_a_training_forward_keeps_repacked_weights_for_the_backwards_that_read_them(T, nf, n, O, B, copy):
    plan = dmt.dmt_plan_create([10] * (T * nf), [n] * (T * nf), "f32", T, [t for t in range(T) for _ in range(nf)], B, 1)
    w = torch.zeros(4)
    params = dmt.make_tm_params([dict(kind="dot_linear", out_dim=O, w_proj=w, b_proj=w)] * T)
    np_pad = -(-(nf * (nf - 1) // 2) // 8) * 8
    up = lambda b: -(-b // 256) * 256
    for dtype, eb in ((torch.bfloat16, 2), (torch.float32, 4)):
        want = T * (up(B * np_pad * eb) + (up(O * (np_pad + nf * n) * eb) if copy and eb == 2 else 0))
        assert dmt.dmt_tm_kept_bytes(plan, params, B, dtype) == want


@pytest.mark.parametrize("T,nf,n,O", [(4, 8, 32, 512), (1, 2, 64, 641), (2, 8, 128, 2048), (4, 3, 64, 1000)])
def test_a_backward_workspace_for_a_larger_batch_serves_a_smaller_one(lib, T, nf, n, O, monkeypatch):
    """Across the line between the two ways of a dot tower's data gradient, whichever way the smaller batch goes."""
    batches = [1, 64, 65, 300, 500, 640, 641, 1024, 2000, 2048, 4096, 8192]
    assert len({one_kernel(lib, T, nf, n, O, B) for B in batches}) == 2

    def sizes(fuse):
        monkeypatch.setenv("DMT_TM_FUSE", fuse)
        plan = dmt.dmt_plan_create([10] * (T * nf), [n] * (T * nf), "f32", T, [t for t in range(T) for _ in range(nf)], 8192, 1)
        w = torch.zeros(4)
        params = dmt.make_tm_params([dict(kind="dot_linear", out_dim=O, w_proj=w, b_proj=w)] * T)
        return [dmt.dmt_tm_bwd_workspace_bytes(plan, params, B) for B in batches]

    either = [sizes(fuse) for fuse in "012"]
    for small in either:
        assert all(a <= b for a, b in zip(small, sizes("1")[1:])), (small, sizes("1"))


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


def test_lds_beyond_the_default_is_asked_for_on_every_device(lib):
    """All kernels with more dynamic LDS than a device grants by itself go through dmt_allow_lds."""
    assert [lib.allow_lds(d, 0) for d in (0, 0, 1, 0, 1, 5)] == [1, 0, 1, 0, 0, 1]
    assert [lib.allow_lds(3, 1), lib.allow_lds(3, 0), lib.allow_lds(3, 0)] == [1, 1, 0]      # a failure is tried again
    uses = {}
    for name in sorted(os.listdir(hip_build.CSRC)):
        with open(os.path.join(hip_build.CSRC, name)) as f:
            n = f.read().count("hipFuncSetAttribute(")
        if n:
            uses[name] = n
    assert uses == {"dmt_internal.h": 1}


# (towers, rows, columns, K of the first segment, of the second, contractions a group stands for) of launches that one
# block per CU works through; tests/test_gpu_tm_forms.py runs them
ONE_BLOCK_PER_CU = [
    (4, 10233, 520, 120, 1024, 0), (4, 10233, 516, 120, 1024, 0), (4, 10233, 520, 66, 768, 0),    # dot terms | pooled values
    (4, 10233, 256, 264, 64, 4), (4, 10233, 256, 264, 24, 4),                                     # a per-feature layer's
    (3, 5900, 1288, 0, 1024, 0), (3, 8200, 2056, 0, 128, 0), (4, 32760, 256, 0, 1024, 0),         # one segment
]


@pytest.mark.parametrize("n,M,N,K0,K1,reps", ONE_BLOCK_PER_CU)
def test_launches_that_one_block_per_cu_works_through(lib, n, M, N, K0, K1, reps):
    tiles = ctypes.c_long()
    assert lib.blocks_of(n, M, N, K0, K1, reps, ctypes.byref(tiles)) == 256 and tiles.value > 256


@pytest.mark.parametrize("n,M,N,K0,K1,reps", [(4, 8192, 512, 0, 1024, 0),                     # a tile a block
                                              (3, 8200, 2056, 0, 64, 0),                      # one K step
                                              (4, 8205, 520, 120, 1024, 0)])                  # many slots without a tile
def test_launches_that_get_a_block_for_every_tile(lib, n, M, N, K0, K1, reps):
    tiles = ctypes.c_long()
    blocks = lib.blocks_of(n, M, N, K0, K1, reps, ctypes.byref(tiles))
    assert blocks >= tiles.value and blocks % 8 == 0


BIAS, CROSS, F32 = 0, 2, 3           # what a launch's outputs are (EPI_*)


@pytest.mark.parametrize("n,M,N,K,dK,epi,dots,tile", [
    (4, 512, 256, 1024, 0, BIAS, 0, 32), (4, 513, 256, 1024, 0, BIAS, 0, 128),            # 512 small tiles and more
    (4, 192, 1024, 1024, 0, CROSS, 0, 32), (4, 193, 1024, 1024, 0, CROSS, 0, 128),        # 768 of cross layers
    (8, 512, 256, 1024, 0, BIAS, 1, 32), (8, 513, 256, 1024, 0, BIAS, 1, 128),            # 1024 with dot terms
    (8, 4096, 256, 1024, 0, BIAS, 0, 128), (8, 4097, 256, 1024, 0, BIAS, 0, 256),         # 512 mid tiles and more
    (8, 4097, 256, 1024, 0, BIAS, 1, 256), (8, 4097, 256, 1024, 64, BIAS, 0, 128),        # ... unequal K
    (8, 4097, 256, 64, 0, BIAS, 0, 128), (8, 4097, 256, 1024, 0, F32, 0, 128),            # ... one K step, gradients
    (4, 1280, 2048, 2048, 0, CROSS, 0, 128), (4, 1281, 2048, 2048, 0, CROSS, 0, 256),     # 192 big tiles
    (8, 6000, 256, 1024, 64, BIAS, 0, 256), (8, 60000, 128, 1024, 0, BIAS, 0, 128),       # ... unless narrow
])
def test_which_tiles_a_launch_takes(lib, n, M, N, K, dK, epi, dots, tile):
    assert lib.forward_tile(n, M, N, K, dK, epi, dots) == tile
