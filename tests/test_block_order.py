"""Host model of the order in which the per-head kernels' workgroups take (head, block) pairs (CPU only): every pair is taken
exactly once, by a workgroup of the head's die where the heads divide over the dies, and the groups of heads that are walked
together differ by one head at most."""
import pytest

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
