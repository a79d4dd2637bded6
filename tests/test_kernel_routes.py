"""Which kernels calls take, and what these can reach (CPU only).  The library is run against a HIP runtime that only
notes what is asked of it."""
import ctypes
import json
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2501_09767_amd", "liblemo_hip.so")

RUNTIME = r"""
#include <stddef.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
static struct { const void* kernel; const char* name; } known[4096];
static int n_known;
static dim3 grid, block;
static size_t lds;
static void* stream;
const char* launched[64];
int threads[64], blocks[64], n_launched;
void** __hipRegisterFatBinary(const void* data) { (void)data; return (void**)known; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* f, char* a, const char* name, unsigned n, void* t, void* b, dim3* bd, dim3* gd, int* w) {
    (void)m; (void)a; (void)n; (void)t; (void)b; (void)bd; (void)gd; (void)w;
    if (n_known < 4096) { known[n_known].kernel = f; known[n_known++].name = strdup(name); }
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, void* s) { grid = g; block = b; lds = l; stream = s; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, void** s) { *g = grid; *b = block; *l = lds; *s = stream; return 0; }
int hipFuncSetAttribute(const void* f, int what, int bytes) { (void)f; (void)what; (void)bytes; return 0; }
int hipGetLastError(void) { return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t l, void* s) {
    (void)args; (void)l; (void)s;
    for (int i = 0; i < n_known && n_launched < 64; ++i)
        if (known[i].kernel == f) { launched[n_launched] = known[i].name; blocks[n_launched] = (int)g.x; threads[n_launched++] = (int)b.x; }
    return 0;
}
"""
P = 1 << 20  # in the place of device addresses: nothing is read
F32, BF16 = 0, 1
CAUSAL = 1
LONGEST = {F32: (1 << 22) - 4, BF16: (1 << 22) - 8}  # token pitch, elements


def run(runtime):
    """In a process of its own: calls from standard input, the kernels each of them launched to standard output."""
    hip = ctypes.CDLL(runtime, mode=ctypes.RTLD_GLOBAL)
    lib = ctypes.CDLL(LIB)
    kinds = {"p": ctypes.c_void_p, "i": ctypes.c_int32, "l": ctypes.c_int64, "f": ctypes.c_float, "z": ctypes.c_size_t}
    for fn, args in (("score_rowstats", "ppliiiillllfipp"), ("score_colsums", "ppliiiillllfiipppp"), ("score_blocks", "ppliiiillllfiiippppzp"),
                     ("select_topk", "pliipp"), ("gather_gemm", "pllplplppliiip"), ("gather_gemm_dx", "pllplpllpiiip"), ("gather_gemm_dw", "plpllplpliiipzp")):
        getattr(lib, "lemo_" + fn).argtypes = [kinds[k] for k in args]
    seen = ctypes.c_int.in_dll(hip, "n_launched")
    names, threads = (ctypes.c_char_p * 64).in_dll(hip, "launched"), (ctypes.c_int * 64).in_dll(hip, "threads")

    def sweeps(dt, d, S, H, flags, q_pitch, k_pitch):
        return lib.lemo_score_rowstats(P, P, S, H, H, d, dt, q_pitch, d, k_pitch, d, 0, flags, P, None) or \
            lib.lemo_score_colsums(P, P, S, H, H, d, dt, q_pitch, d, k_pitch, d, 0, 128, flags, P, P, P, None)

    def blocks(dt, d, S, H, flags):
        return lib.lemo_score_blocks(P, P, S, H, H, d, dt, H * d, d, H * d, d, 0, 64, flags, 0, P, None, P, P, 1 << 40, None)

    def topk(S, L):
        return lib.lemo_select_topk(P, S, L, max(1, L // 3), P, None)

    def gemm(dt, M, N, K):
        return lib.lemo_gather_gemm(P, M, K, None, M, P, K, None, P, N, K, N, dt, None)

    def gemm_dx(dt, M, N, K):  # [M, N], contraction K
        return lib.lemo_gather_gemm_dx(P, K, M, P, N, P, N, M, None, N, K, dt, None)

    def gemm_dw(dt, M, N, K):  # [M, N] of K tokens
        return lib.lemo_gather_gemm_dw(P, M, P, K, N, None, K, 1 << 50, N, N, M, dt, P, 1 << 40, None)

    out = []
    for entry, *args in json.load(sys.stdin):
        seen.value = 0
        rc = {"sweeps": sweeps, "blocks": blocks, "topk": topk, "gemm": gemm, "gemm_dx": gemm_dx, "gemm_dw": gemm_dw}[entry](*args)
        assert rc == 0, (entry, args, rc)
        out.append([(names[i].decode(), threads[i]) for i in range(seen.value)])
    json.dump(out, sys.stdout)


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """calls (entry, arguments) -> per call the names of the kernels it launched and their workgroups' threads"""
    source = tmp_path_factory.mktemp("runtime") / "runtime.c"
    runtime = source.with_suffix(".so")
    source.write_text(RUNTIME)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(source), "-o", str(runtime)], check=True)

    def ask(calls):
        r = subprocess.run([sys.executable, __file__, str(runtime)], input=json.dumps(calls), capture_output=True, text=True)
        assert r.returncode == 0, r.stdout + r.stderr
        return json.loads(r.stdout)
    return ask


@pytest.fixture
def routes(launches):
    """calls (type, head size, tokens, heads, flags, pitch of Q, of K) -> per call the (D, NRT, KS, WAVES, binary32) of its sweeps"""
    def ask(calls):
        out = []
        for made in launches([("sweeps", *c) for c in calls]):
            assert len(made) == 2
            kinds = []
            for sweep, (name, threads) in zip(("rowstats", "colsum"), made):
                m = re.search(sweep + r"(_f32)?_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", name)
                assert m, name
                kinds.append((*(int(m[i]) for i in range(2, 6)), m[1] is not None))
                assert threads == 64 * kinds[-1][3]
            out.append(kinds)
        return out
    return ask


def sizes():
    """Tokens and heads over the ranges of all rules that choose a kernel."""
    tokens = (300, 384, 500, 512, 700, 1024, 1500, 2048, 3000, 4096, 5000, 8192, 12345, 14336, 16384, 32768)
    return [(S, H) for S in tokens for H in (1, 2, 3, 4, 5, 7, 8, 9, 11, 12, 14, 16, 20, 24, 28, 32, 40, 64, 128)]


@pytest.mark.parametrize("dt,d", [(dt, d) for dt in (F32, BF16) for d in (64, 128)])
def test_stages_are_within_reach_at_every_pitch(routes, dt, d):
    """The offset of a row in a stage and the size of the stage's descriptor have 31 bits: rows beyond would arrive as zeros."""
    size = 4 if dt == F32 else 2
    calls, longest = [], 0
    for S, H in sizes():
        for flags in (0, CAUSAL):
            for q, k in ((LONGEST[dt], LONGEST[dt]), (d, LONGEST[dt]), (LONGEST[dt], d), (1 << 20, 1 << 20)):
                calls.append((dt, d, S, H, flags, q, k))
    for call, kinds in zip(calls, routes(calls)):
        for D, nrt, ks, waves, f32 in kinds:
            assert D == d and f32 == (dt == F32)
            rows, row_bytes = (64 if d * size > 256 else 128) * waves // 4, max(call[5:]) * size
            reach = (rows - 1) * row_bytes + d * size
            assert reach <= 0x7fffffff, (call, kinds)
            longest = max(longest, reach)
    assert longest > 1 << 30


@pytest.mark.parametrize("d,most", [(64, 1024), (128, 640)])
def test_shared_rows_stay_shared(routes, d, most):
    """Waves that share rows add up stage by stage and round the row statistics once: column sums of 14336 tokens, 16 heads of 64 are
    7e-8 from 64 bits where waves with rows of their own are 1.2e-6 off.  Launches that were small enough for the former keep them."""
    calls = [(BF16, d, S, H, flags, H * d, H * d) for S, H in sizes() for flags in (0, CAUSAL)]
    shared = 0
    for call, kinds in zip(calls, routes(calls)):
        S, H, flags = call[2:5]
        n = H * ((S + 255) // 256)                            # blocks of 256 rows
        if n <= most and (flags & CAUSAL or n <= 64 or (2 * n + 255) // 256 % 2 == 1):
            shared += 1
            assert all(k[2] > 1 for k in kinds), (call, n, kinds)
    assert shared > 200


@pytest.mark.parametrize("dt,d,S,H,causal,ks,waves", [
    # many heads of few tokens under the mask
    (BF16, 128, 1500, 20, 1, 4, 4), (BF16, 128, 2048, 16, 1, 4, 4), (BF16, 128, 1024, 64, 1, 2, 4), (BF16, 128, 1323, 36, 1, 2, 4), (BF16, 128, 2048, 64, 1, 2, 4),
    (BF16, 128, 1846, 56, 1, 2, 4), (BF16, 128, 4096, 64, 1, 1, 4),
    # a last round that blocks of 512 rows would leave nearly empty
    (BF16, 128, 5376, 48, 1, 1, 4), (BF16, 128, 2304, 112, 0, 1, 4), (BF16, 128, 6254, 40, 0, 1, 4), (BF16, 64, 5376, 48, 0, 1, 4), (BF16, 64, 5376, 24, 0, 1, 4),
    # a last stage that is half empty
    (BF16, 128, 640, 16, 0, 4, 4), (BF16, 64, 513, 20, 0, 4, 4), (BF16, 64, 640, 32, 0, 2, 4), (BF16, 128, 640, 64, 0, 1, 4), (F32, 64, 384, 4, 0, 4, 4), (F32, 64, 384, 4, 1, 4, 4),
    # and where eight waves are the faster ones
    (BF16, 128, 512, 16, 0, 8, 8), (BF16, 128, 641, 16, 0, 8, 8), (BF16, 128, 513, 16, 1, 8, 8), (BF16, 128, 1949, 14, 1, 8, 8), (BF16, 128, 1500, 32, 1, 4, 8),
    (BF16, 128, 4096, 32, 1, 2, 8), (BF16, 128, 8192, 32, 1, 1, 8), (BF16, 128, 8192, 32, 0, 1, 8), (BF16, 64, 8192, 16, 0, 1, 8), (F32, 64, 385, 4, 1, 8, 8)])
def test_eight_waves_only_where_they_are_faster(routes, dt, d, S, H, causal, ks, waves):
    """Calls on either side of the rules' lines, each with the kernel that was measured to be the faster one."""
    for _, _, k, w, _ in routes([(dt, d, S, H, causal, H * d, H * d)])[0]:
        assert (k, w) == (ks, waves)


def test_the_shapes_of_the_eight_wave_tests_take_them(routes):
    from test_gpu_parity import EIGHT_WAVES
    calls = [(F32 if dt == "f32" else BF16, d, S, H, flags & CAUSAL, H * d, H * d) for S, H, _, d, flags, dt in EIGHT_WAVES]
    taken = set()
    for call, kinds in zip(calls, routes(calls)):
        assert all(k[3] == 8 for k in kinds), (call, kinds)
        taken.add((call[0], call[1], call[4], kinds[0][2]))
    assert taken == {(BF16, 128, c, ks) for c in (0, 1) for ks in (8, 4, 2, 1)} | {(BF16, 64, 1, 8)} | {(BF16, 64, 0, ks) for ks in (8, 4, 1)} | \
        {(F32, 64, c, 8) for c in (0, 1)} | {(F32, 128, c, 4) for c in (0, 1)}


@pytest.mark.parametrize("d,S,H,causal,first", [
    # 65 to 128 rectangles: quarters from 20 heads of 128 on, and for all of 64
    (128, 1200, 1, 0, "tilemax_kernel"), (128, 1500, 4, 1, "tilemax_kernel"), (128, 1800, 16, 1, "tilemax_kernel"), (128, 1800, 20, 1, "tilemax_few_kernel"),
    (128, 1200, 32, 0, "tilemax_few_kernel"), (64, 1800, 1, 1, "tilemax_few_kernel"), (64, 1408, 4, 0, "tilemax_few_kernel"),
    # up to 64, and more than 128
    (128, 1000, 1, 0, "tilemax_few_kernel"), (128, 1921, 32, 1, "tilemax_kernel"), (64, 1921, 4, 1, "tilemax_kernel")])
def test_rectangles_in_quarters_only_where_they_are_faster(launches, d, S, H, causal, first):
    names = [name for name, _ in launches([("blocks", BF16, d, S, H, causal)])[0]]
    assert len(names) == 2 and re.match(r"_ZN4lemo\d+" + first, names[0]), names


@pytest.mark.parametrize("S,L,threads", [(32768, 16, 256), (32768, 128, 256), (32768, 129, 512), (100, 4096, 256), (4096, 2048, 512), (4096, 2049, 1024), (32768, 32768, 1024)])
def test_threads_of_a_selection(launches, S, L, threads):
    """Short segments on few threads: on 512, all scores equal, they were slower than with digits of 8 bits."""
    (name, n), = launches([("topk", S, L)])[0]
    assert "select_topk_kernel" in name and n == threads


@pytest.mark.parametrize("entry", ["gemm", "gemm_dw"])
@pytest.mark.parametrize("M,N,edge", [(16, 16, 16), (256, 512, 16), (512, 256, 16), (260, 512, 32), (368, 512, 32), (256, 768, 32), (192, 1024, 32), (800, 256, 32)])
def test_small_fp32_tiles(launches, entry, M, N, edge):
    """16 x 16 tiles up to two per CU (512), 32 x 32 ones beyond."""
    for K in (16, 1024):
        names = [name for name, _ in launches([(entry, F32, M, N, K)])[0]]
        assert len(names) == 1 and re.search(r"gather_gemm_small_kernelIfLb[01]ELi\dELi1ELi1ELb0ELi(\d+)E", names[0])[1] == str(edge), names


@pytest.mark.parametrize("entry,M,N,K,tile", [
    ("gemm_dx", 100, 512, 512, "64x64"), ("gemm_dx", 408, 512, 512, "64x64"), ("gemm_dx", 2000, 512, 512, "64x64"), ("gemm_dx", 3277, 512, 512, "64x128"),
    ("gemm_dx", 256, 256, 256, "64x128"), ("gemm_dx", 256, 256, 768, "64x64"), ("gemm_dx", 2000, 768, 768, "64x128"),
    ("gemm", 50, 256, 256, "64x128"), ("gemm", 5000, 256, 256, "64x128"), ("gemm", 408, 512, 512, "64x128"), ("gemm", 256, 256, 1024, "64x64"), ("gemm", 408, 3072, 768, "64x128")])
def test_tiles_of_narrow_bf16_products(launches, entry, M, N, K, tile):
    """64 x 64 tiles against 64 x 128 ones, which cost an input gradient more: the one that was measured to be faster."""
    names = [name for name, _ in launches([(entry, BF16, M, N, K)])[0]]
    assert len(names) == 1 and re.search({"64x64": "gather_gemm_small_kernel", "64x128": r"gather_gemm_mid_kernelILb[01]ELi\dELi1E"}[tile], names[0]), names


def test_the_shapes_of_the_tile_tests_take_their_kinds(launches):
    from test_gpu_parity import TILE_KINDS
    kernel = {"256x256": "large_kernel", "256x128": r"mid_kernelILb[01]ELi\dELi4E", "192x128": r"mid_kernelILb[01]ELi\dELi3E", "128x128": r"mid_kernelILb[01]ELi\dELi2E",
              "64x128": r"mid_kernelILb[01]ELi\dELi1E", "64x64": "small_kernel"}
    entry = {"nt": "gemm", "add": "gemm", "dx": "gemm_dx"}   # (the in-place add takes the tiles of the plain product)
    for kind, shapes in TILE_KINDS.items():
        assert {entry[form] for form, *_ in shapes} == {"gemm", "gemm_dx"}
        for shape, made in zip(shapes, launches([(entry[form], BF16, *size) for form, *size in shapes])):
            assert len(made) == 1 and re.search(kernel[kind], made[0][0]), (kind, shape, made)


if __name__ == "__main__":
    run(sys.argv[1])
