"""The order in which workgroups take their work (CPU only).  Host model of the order in which the per-head kernels' workgroups take (head, block) pairs (CPU only): every pair is taken
exactly once, by a workgroup of the head's die where the heads divide over the dies, and the groups of heads that are walked
together differ by one head at most."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DIES = 8


def head_order(H, causal, limit):
    per_die = H // DIES if H % DIES == 0 else 0
    heads, together = per_die or H, (limit if causal else 1) * (1 if per_die else DIES)
    return per_die, -(-heads // together) if heads < 1 << 15 else 1


def decode_block(b, H, nblk, per_die, groups):
    x, w, heads = (b % DIES, b // DIES, per_die) if per_die else (0, b, H)
    first, width = 0, heads
    if groups > 1:
        g = ((w // nblk + 1) * groups - 1) // heads
        first = g * heads // groups
        width = (g + 1) * heads // groups - first
    r = w - first * nblk
    return x * per_die + first + r % width, r // width, width


@pytest.mark.parametrize("nblk", [1, 2, 7, 33])
@pytest.mark.parametrize("causal,limit", [(False, 8), (True, 1), (True, 2), (True, 8), (True, 64)])
def test_every_block_of_every_head_once(nblk, causal, limit):
    for H in list(range(1, 100)) + [100, 128, 257, 320]:
        per_die, groups = head_order(H, causal, limit)
        taken = [decode_block(b, H, nblk, per_die, groups) for b in range(H * nblk)]
        assert {(h, r) for h, r, _ in taken} == {(h, r) for h in range(H) for r in range(nblk)}
        assert max(w for _, _, w in taken) - min(w for _, _, w in taken) <= 1
        if per_die:
            assert all(h // per_die == b % DIES for b, (h, _, _) in enumerate(taken))
        assert groups < 1 << 15 and (per_die or H) < 1 << 16  # the kernel's products fit 32 bits


RECTANGLES = r"""
#include <math.h>
#include <stdio.h>
#include <vector>
#include "score_blocks.hpp"
using namespace lemo;
// ids 0 .. total - 1 of the order, or the last `tail` of them: inside the matrix, on or below the diagonal, each once, bands of four
// rows from the top, a band column by column
static int check(int nt, bool causal, long long tail) {
    const long long total = causal ? (long long)nt * (nt + 1) / 2 : (long long)nt * nt, first = tail < total ? total - tail : 0;
    std::vector<char> seen(first == 0 ? (size_t)nt * nt : 0);
    int q = -1, k = -1;
    for (long long id = first; id < total; ++id) {
        int tq = -1, tk = -1;
        sb_rectangle((int)id, nt, causal, tq, tk);
        if (tq < 0 || tq >= nt || tk < 0 || tk >= nt || (causal && tk > tq)) return printf("nt %d causal %d: %lld at %d, %d\n", nt, causal, id, tq, tk), 1;
        if (id > first && !(tq / 4 > q / 4 || (tq / 4 == q / 4 && (tk > k || (tk == k && tq == q + 1))))) return printf("nt %d causal %d: %lld out of order\n", nt, causal, id), 1;
        if (!seen.empty() && seen[(size_t)tq * nt + tk]++) return printf("nt %d causal %d: %d, %d twice\n", nt, causal, tq, tk), 1;
        q = tq;
        k = tk;
    }
    return q != nt - 1 || k != nt - 1;  // the last one
}
int main() {
    for (int causal = 0; causal < 2; ++causal) {
        for (int nt = 1; nt <= 130; ++nt)
            if (check(nt, causal, 1ll << 40)) return 1;
        for (int nt : {255, 256, 257, 1000, 4097, 16384, 32767})  // 4 million tokens; the root of the band is taken in binary32
            if (check(nt, causal, 1000)) return 1;
    }
    return 0;
}
"""


def test_rectangles_of_block_scores(tmp_path):
    """sb_rectangle itself, compiled for the host."""
    source, program = tmp_path / "rectangles.hip", tmp_path / "rectangles"
    source.write_text(RECTANGLES)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2501_09767_amd", "csrc"), str(source), "-o", str(program)], check=True, capture_output=True)
    r = subprocess.run([str(program)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
