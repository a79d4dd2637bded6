"""Host model of the loads and LDS positions of the selective-load GEMM on tiles of 256 x 256 and of 256, 192, 128 or 64 x 128 (CPU only).

An operand's slab comes in regions of 128 rows (contraction-major: 64 rows of 128 columns); a 256-wide tile has two of them.
Unit u of a region (16 bytes) goes to its LDS bytes [16 u, 16 u + 16), and the lane that asks for it chooses which piece of
which row that is.  This restates the kernel's formulas and its order of loads and reads, and checks that every request the
range check lets through stays inside its operand, that the fragment reads find the piece they want, and that no region is
read before its load was waited for or loaded again before its reads were."""
import itertools

import pytest

KB, THREADS, NLD, TA, TB = 128, 512, 2, 4, 2


def kswz(r):
    return ((r & 3) | ((r >> 3) & 1) << 2) << 1


def unit(i, tid):
    """(row, byte) of unit i * THREADS + tid: rows along the contraction, contraction-major rows."""
    krow = tid >> 4
    return ((i * (THREADS // 8) + (tid >> 3), ((tid & 7) ^ ((tid >> 4) & 7)) * 16),
            (i * (THREADS // 16) + krow, ((tid & 15) ^ kswz(krow)) * 16))


def test_fragments_find_their_pieces():
    along, across = {}, {}
    for i in range(NLD):
        for tid in range(THREADS):
            along[i * THREADS + tid], across[i * THREADS + tid] = unit(i, tid)
    assert sorted(along.values()) == [(r, 16 * p) for r in range(128) for p in range(8)]
    assert sorted(across.values()) == [(r, 16 * p) for r in range(64) for p in range(16)]
    for t in range(8):                                       # 16-row tiles of a region
        for c in range(2):
            banks = {}
            for lane in range(64):
                l16, quad = lane & 15, lane >> 4
                at = t * 16 * KB + l16 * KB + (((4 * c + quad) ^ ((l16 >> 1) & 7)) << 4)
                assert along[at // 16] == (t * 16 + l16, (4 * c + quad) * 16)
                banks.setdefault(quad, set()).add(at // 16 % 16)
                trow = 8 * quad + (l16 >> 2)
                for step in (0, 4):                          # the two transposing reads: four columns of row `trow`
                    at = trow * 256 + (lane & 1) * 8 + c * 32 * 256 + (((t * 2 + ((lane & 3) >> 1)) ^ kswz(trow)) << 4) + step * 256
                    col = t * 16 + (lane & 3) * 4
                    assert across[at // 16] == (c * 32 + trow + step, col * 2 // 16 * 16) and at % 16 == col * 2 % 16
            assert all(len(b) == 16 for b in banks.values())


def requests(layout, bm, bn, M, N, K, S, lda, ldb, idx):
    """(operand, base, size, offset checked, scalar offset, row, byte in the row, wanted)"""
    kbytes, nk = K * 2, -(-K // 64)
    a_rows = K if layout == "tn" else S
    a_bytes, b_bytes = ((a_rows - 1) * lda + (M if layout == "tn" else K)) * 2, ((S - 1) * ldb + N) * 2
    for m0, n0 in itertools.product(range(0, M, bm), range(0, N, bn)):
        for kt in list(range(nk)) + [nk, nk + 3]:            # the loops ask for up to four slabs past the end
            live = kt < nk
            for i, tid in itertools.product(range(NLD), (0, 1, 7, 8, 130, 511)):
                (row, kpos), (krow, kcol) = unit(i, tid)
                in_k, k = kpos < kbytes - kt * KB, kt * 64 + krow
                for r in range(-(-bm // 128)):
                    if r * 2 + i >= bm // 64:                # the kinds of 64 and 192 rows end with half a region
                        continue
                    if layout == "tn":
                        off = kt * 64 * lda * 2 if live else 0
                        yield ("A", m0 * 2 + off, ((K - 1) * lda + M - m0) * 2 - off if live else 0, krow * lda * 2 + r * 256 + kcol, 0, k,
                               m0 * 2 + r * 256 + kcol, k < K)
                    else:
                        m = min(m0 + r * 128 + row, M - 1)
                        a_row = idx[m] if layout == "nt" else m
                        yield "A", 0, a_bytes, a_row * lda * 2 + kpos if in_k else a_bytes, kt * KB, a_row, kt * KB + kpos, in_k
                for r in range(bn // 128):
                    if layout == "tn":
                        tok = idx[k] * ldb * 2 if k < K else b_bytes
                        yield ("B", 0, b_bytes, tok if tok == b_bytes else tok + n0 * 2 + r * 256 + kcol, 0, idx[k] if k < K else 0,
                               n0 * 2 + r * 256 + kcol, k < K)
                    elif layout == "nt":
                        size = (min(bn, N - n0) - 1) * ldb * 2 + kbytes
                        yield ("B", n0 * ldb * 2, size, (r * 128 + row) * ldb * 2 + kpos if in_k else size, kt * KB, n0 + r * 128 + row, kt * KB + kpos,
                               in_k and n0 + r * 128 + row < N)
                    else:
                        off = kt * 64 * ldb * 2 if live else 0
                        yield ("B", n0 * 2 + off, ((K - 1) * ldb + N - n0) * 2 - off if live else 0, krow * ldb * 2 + r * 256 + kcol, 0, k,
                               n0 * 2 + r * 256 + kcol, k < K)


@pytest.mark.parametrize("layout,M,N,K,pad", [("nt", 300, 270, 72, 0), ("nt", 1, 1, 8, 8), ("nt", 257, 513, 200, 16), ("nn", 260, 264, 72, 0),
                                              ("nn", 300, 512, 200, 8), ("tn", 264, 520, 65, 0), ("tn", 256, 264, 131, 8), ("tn", 8, 8, 1, 0), ("nt", 130, 40, 1000, 0), ("nt", 517, 300, 256, 8),
                                              ("nt", 513, 257, 1000, 0), ("nt", 1, 2, 8, 0), ("nt", 300, 512, 4096, 0), ("nt", 256, 256, 64, 24)])
@pytest.mark.parametrize("bm,bn", [(256, 256), (256, 128), (128, 128), (192, 128), (64, 128)])
def test_no_request_leaves_its_operand(layout, M, N, K, pad, bm, bn):
    S = (K if layout == "tn" else M) + (0 if layout == "nn" else 9)
    idx = [(7 * r + 3) % S for r in range(K if layout == "tn" else M)]
    lda, ldb = (M if layout == "tn" else K) + pad, (K if layout == "nt" else N) + pad
    width = {"A": M if layout == "tn" else K, "B": K if layout == "nt" else N}
    total = {"A": (((K if layout == "tn" else S) - 1) * lda + width["A"]) * 2, "B": (({"nt": N, "nn": K, "tn": S}[layout] - 1) * ldb + width["B"]) * 2}
    for op, base, size, voff, soff, row, byte, wanted in requests(layout, bm, bn, M, N, K, S, lda, ldb, idx):
        if voff + soff + 16 <= size:                         # the hardware lets it through
            assert 0 <= base + voff + soff <= total[op] - 16, (op, base, size, voff, soff)
        if wanted and byte + 16 <= width[op] * 2:
            assert voff + soff + 16 <= size and base + voff + soff == row * (lda if op == "A" else ldb) * 2 + byte, (op, row, byte)
        if not wanted:
            assert voff >= size, (op, row, byte)             # arrives as zeros


@pytest.mark.parametrize("nk", [1, 2, 3, 6])
@pytest.mark.parametrize("tn", [False, True])
def test_regions_are_waited_for_and_free(nk, tn):
    """256 x 256 tiles.  One wave's order of loads, waits and reads; a barrier makes what every wave has waited for true of all of them.
    Weight gradient: the kept rows' indices of a slab come through a ring of four entries (the wave's own) into registers, from
    which the loads of B take them."""
    events = []                                              # loads in issue order: (region, slab), one entry per load
    place = lambda reg, kt: (reg, kt & 1)                    # where a region of a slab lies
    holds, unread = {}, {}
    entry, tokens = {n: n for n in range(4)}, None           # (the first four entries are waited for before anything else)

    def load(reg, kt):
        p = place(reg, kt)
        assert not unread.get(p), (reg, kt, "overwrites fragments still to be read")
        if tn and reg[0] == "B":
            assert tokens == kt, (reg, kt, "rows of another slab")
        for _ in range(NLD):
            events.append((p, kt))
        holds[p], unread[p] = kt, True

    def landed(what, published):
        return max(n for n, e in enumerate(events) if e == what) < published

    def read(reg, kt, published):
        p = place(reg, kt)
        assert holds[p] == kt and landed((p, kt), published), (reg, kt)

    def read_tokens(kt, published):
        nonlocal tokens
        if tn:
            assert entry[kt % 4] == kt and (kt < 4 or landed(("tokens", kt), published)), (kt, "indices")
            tokens = kt

    for step in (0, ("B0", 0), ("A0", 0), ("B1", 0), ("A1", 0), 1, ("B1", 1), ("A0", 1), ("B0", 1), 2):
        load(*step) if isinstance(step, tuple) else read_tokens(step, 0)
    published = len(events) - 5 * NLD
    late = []                                                # read in the quarter before: awaited by the next barrier but one
    for reg in ("B0", "A0"):
        read(reg, 0, published)
        unread[place(reg, 0)] = False                        # (all fragments awaited before the loop)
    for kt in range(nk):
        F, L = ("B0", "B1") if kt % 2 == 0 else ("B1", "B0")
        published = len(events) - 3 * NLD
        for q1, q2, loads in (((L, kt), ("A1", kt), [("A1", kt + 1), (F, kt + 2)]), ((L, kt + 1), ("A0", kt + 1), [("A0", kt + 2), (L, kt + 2)])):
            done, late = late, []
            for p in done:
                unread[p] = False
            if tn and q2[0] == "A0":
                assert entry[kt % 4] == kt                   # (its indices were read three slabs ago)
                events.append(("tokens", kt + 4))
                entry[kt % 4] = kt + 4
            for reg, s in loads:
                load(reg, s)
            read(*q1, published)
            if q2[0] == "A0":
                read_tokens(kt + 3, published)
            read(*q2, published)
            # at the next barrier the first quarter's reads are awaited, the second's only at the one after
            unread[place(*q1)] = False
            late = [place(*q2)]
            published = len(events) - 3 * NLD


@pytest.mark.parametrize("nk", [1, 2, 3, 4, 5, 9])
@pytest.mark.parametrize("ua,stages,tn", [(1, 4, False), (2, 4, False), (2, 4, True), (3, 4, False), (4, 3, False), (4, 3, True)])
def test_ring_is_waited_for_and_free(nk, ua, stages, tn):
    """Tiles of 64 ua x 128: slabs in a ring of stages, and the kept rows' indices in a ring of four entries."""
    batch, ahead = ua + NLD + tn, stages - 1
    events, holds, unread, entry = [], {}, {}, {}

    def done(what, outstanding):                              # loads complete in issue order
        return max(n for n, e in enumerate(events) if e == what) < len(events) - outstanding

    def load(kt):
        assert not unread.get(kt % stages), (kt, "overwrites fragments still to be read")
        if tn:
            assert entry[kt % 4] == kt, (kt, "indices of another slab")
        events.extend([("slab", kt)] * (ua + NLD))
        holds[kt % stages], unread[kt % stages] = kt, True
        if tn:
            events.append(("idx", kt + ahead))
            entry[(kt + ahead) % 4] = kt + ahead

    if tn:
        entry = {n: n for n in range(4)}                      # waited for before the first rows
    for kt in range(stages):
        load(kt)
    assert done(("slab", 0), (stages - 1) * batch)
    unread[0] = False                                         # slab 0's fragments are read
    for kt in range(nk):
        outstanding = (stages - 2) * batch
        assert done(("slab", kt + 1), outstanding) and holds[(kt + 1) % stages] == kt + 1
        if tn and ("idx", kt + stages) in events:
            assert done(("idx", kt + stages), outstanding)
        load(kt + stages)
        unread[(kt + 1) % stages] = False                     # read during this step, awaited before the next barrier
