"""An entry point raises the dynamic-LDS limits of all its kernels in its first call for a type and head size, whatever kernel that call
takes itself: a stream capture may then hold calls of any size.  The library is run against a HIP runtime that only notes
what is asked of it, so that no GPU is needed."""
import ctypes
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2501_09767_amd", "liblemo_hip.so")

RUNTIME = r"""
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim3;
struct event { const void* kernel; long bytes; int launch; };
struct event events[1 << 16];
int n_events;
static void note(const void* kernel, long bytes, int launch) {
    if (n_events < 1 << 16) events[n_events++] = (struct event){kernel, bytes, launch};
}
static dim3 grid, block;
static size_t lds;
static void* stream;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, void* s) { grid = g; block = b; lds = l; stream = s; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, void** s) { *g = grid; *b = block; *l = lds; *s = stream; return 0; }
int hipFuncSetAttribute(const void* f, int what, int bytes) { (void)what; note(f, bytes, 0); return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t l, void* s) { (void)g; (void)b; (void)args; (void)s; note(f, (long)l, 1); return 0; }
int hipGetLastError(void) { return 0; }
"""
PLAIN = 64 << 10           # a launch may ask for as much without further ado
P, FAR = 1 << 20, 1 << 50  # in the place of device addresses: nothing is read
F32, BF16 = 0, 1


SIZES = [(1, 1), (300, 4), (300, 12), (1024, 4), (1000, 32), (3000, 32), (6001, 16), (5000, 100), (32768, 32)]  # tokens, heads
PRODUCTS = [(1, 8, 8), (200, 4096, 4096), (1504, 4096, 4096), (3280, 11008, 4096), (700, 1304, 72), (3000, 4096, 4096), (9000, 8192, 8192), (600, 11008, 4096)]


def score(lib, dt, d):
    for S, H in SIZES:
        for flags in (3, 0):
            yield lib.lemo_score_rowstats, (P, P, S, H, H, d, dt, H * d, d, H * d, d, 0, flags, P, None)


def colsums(lib, dt, d):
    for S, H in SIZES:
        for flags in (3, 0):
            yield lib.lemo_score_colsums, (P, P, S, H, H, d, dt, H * d, d, H * d, d, 0, 128, flags, P, P, P, None)


def blocks(lib, dt, d):
    for S in (2048, 100, 1000, 4096, 300, 32768):
        for mode, lse2 in ((1, None), (0, P), (0, None)):
            for flags in (3, 0):
                yield lib.lemo_score_blocks, (P, P, S, 32, 32, d, dt, 32 * d, d, 32 * d, d, 0, 64, flags, mode, lse2, None, P, P, 1 << 40, None)


def attention(lib, dt, d):
    for M, H in [(100, 4), (1000, 8), (1000, 100), (9000, 32), (300, 64)]:
        for v in (H * d, 2 * H * d):  # V with rows as long as K's, and with others
            yield lib.lemo_kept_attention, (P, P, P, 10000, H, H, d, dt, H * d, d, H * d, d, v, d, P, M, 0, 1, FAR, H * d, d, P, 1 << 40, None)


def gemm(lib, dt, _):
    for M, N, C in PRODUCTS:
        yield lib.lemo_gather_gemm, (P, M, C, None, M, P, C, None, P, N, C, N, dt, None)


def gemm_add(lib, dt, _):
    for M, N, C in PRODUCTS:
        yield lib.lemo_gather_gemm_add, (P, M, C, None, M, P, C, None, P, N, M, None, C, N, dt, None)


def gemm_dx(lib, dt, _):
    for M, C, N in PRODUCTS:
        yield lib.lemo_gather_gemm_dx, (P, N, M, P, C, P, C, M, None, C, N, dt, None)


def gemm_dw(lib, dt, _):
    for N, C, M in PRODUCTS + [(4096, 4096, 2)]:
        N = (N + 7) // 8 * 8
        for dW in (FAR, P) if dt == F32 else (FAR,):  # apart from the operands, and over one of them
            yield lib.lemo_gather_gemm_dw, (P, N, 1 << 45, M, C, None, M, dW, C, C, N, dt, P, 1 << 40, None)


ENTRIES = {"score": (score, [(dt, d) for dt in (F32, BF16) for d in (64, 128)]), "colsums": (colsums, [(dt, d) for dt in (F32, BF16) for d in (64, 128)]),
           "blocks": (blocks, [(dt, d) for dt in (F32, BF16) for d in (64, 128)]), "attention": (attention, [(BF16, 64), (BF16, 128)]),
           "gemm": (gemm, [(F32, 0), (BF16, 0)]), "gemm_add": (gemm_add, [(F32, 0), (BF16, 0)]), "gemm_dx": (gemm_dx, [(BF16, 0)]), "gemm_dw": (gemm_dw, [(F32, 0), (BF16, 0)])}


def run(runtime, name):
    """In a process of its own: the calls of one entry point, the first of which may raise limits."""
    class Event(ctypes.Structure):
        _fields_ = [("kernel", ctypes.c_void_p), ("bytes", ctypes.c_long), ("launch", ctypes.c_int)]
    hip = ctypes.CDLL(runtime, mode=ctypes.RTLD_GLOBAL)
    lib = ctypes.CDLL(LIB)
    kinds = {"p": ctypes.c_void_p, "i": ctypes.c_int32, "l": ctypes.c_int64, "f": ctypes.c_float, "z": ctypes.c_size_t}
    for fn, args in (("score_rowstats", "ppliiiillllfipp"), ("score_colsums", "ppliiiillllfiipppp"), ("score_blocks", "ppliiiillllfiiippppzp"),
                     ("kept_attention", "pppliiiillllllplfipllpzp"), ("gather_gemm", "pllplplppliiip"), ("gather_gemm_add", "pllplplppllpiiip"),
                     ("gather_gemm_dx", "pllplpllpiiip"), ("gather_gemm_dw", "plpllplpliiipzp")):
        getattr(lib, "lemo_" + fn).argtypes = [kinds[k] for k in args]
    seen = ctypes.c_int.in_dll(hip, "n_events")
    events = (Event * (1 << 16)).in_dll(hip, "events")
    for dt, d in ENTRIES[name][1]:
        limits, kernels, late = {}, set(), []
        for i, (call, args) in enumerate(ENTRIES[name][0](lib, dt, d)):
            seen.value = 0
            rc = call(*args)
            assert rc == 0, (name, dt, d, i, rc)
            assert any(events[e].launch for e in range(seen.value))
            for e in range(seen.value):
                ev = events[e]
                if not ev.launch:
                    limits[ev.kernel] = ev.bytes
                    if i > 0:
                        late.append((i, ev.bytes))
                else:
                    kernels.add(ev.kernel)
                    assert ev.bytes <= max(PLAIN, limits.get(ev.kernel, 0))
        print(name, dt, d, "kernels", len(kernels), "limits", len(limits), "late", late)
        assert not late, f"{name}: limits raised in call(s) {late}, after the first"


@pytest.mark.parametrize("name", list(ENTRIES))
def test_limits_are_raised_in_the_first_call(tmp_path, name):
    source, runtime = tmp_path / "runtime.c", tmp_path / "runtime.so"
    source.write_text(RUNTIME)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(source), "-o", str(runtime)], check=True)
    r = subprocess.run([sys.executable, __file__, str(runtime), name], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    run(sys.argv[1], sys.argv[2])
