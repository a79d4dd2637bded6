"""Host model of the loads and LDS positions of the selective-load GEMM on 64 x 64 tiles (bf16), 128 x 128 and 32 x 32 ones (binary32) (CPU only).

The kernel fills its slabs with LDS-direct loads: unit u of an operand's slab (16 bytes) goes to LDS bytes [16 u, 16 u + 16),
and the lane that asks for it chooses which piece of which row that is.  The range check of the buffer descriptor takes
the per-thread and the scalar offset together.  This restates the kernel's formulas, in the three operand layouts, and checks that
every request that passes the check stays inside its operand, that pieces past the end of the contraction are refused in at
least one operand, and that the fragment reads find the piece they want where the loads put it."""
import pytest

KB = 128


class Geo:
    def __init__(self, gw, esz, wt):
        self.gw, self.esz, self.wt = gw, esz, wt
        self.w = 2 if gw == 4 else 1
        self.rows = 32 * wt * self.w                      # rows (or columns) of the output tile
        self.groups = 4 // gw
        self.nld = self.rows * KB // (gw * 1024)
        self.krows = KB // esz
        self.pieces = 2 * wt * self.w * esz

    @staticmethod
    def swz(r):
        return (r >> 1) & 7

    def kswz(self, r):
        if self.wt == 1:
            return 0
        if self.esz == 4:
            return ((r >> 2) & 1) << 3
        return ((r >> 1) & 1) << 2


SHAPES = [(1, 2, 2), (4, 4, 2), (1, 4, 1)]


@pytest.mark.parametrize("gw,esz,wt", SHAPES)
def test_fragments_find_their_pieces(gw, esz, wt):
    g = Geo(gw, esz, wt)
    along, across = {}, {}                                # LDS unit -> (row, piece), rows along the contraction / contraction-major
    for i in range(g.nld):
        for t in range(64 * gw):
            u = i * 64 * gw + t
            row = i * 8 * gw + (t >> 3)
            assert row == u // 8
            along[u] = (row, (t & 7) ^ g.swz(row))
            krow = u // g.pieces
            across[u] = (krow, (u % g.pieces) ^ g.kswz(krow))
    assert sorted(along.values()) == [(r, p) for r in range(g.rows) for p in range(8)]
    assert sorted(across.values()) == [(r, p) for r in range(g.krows) for p in range(g.pieces)]
    for w in range(g.w):
        for i in range(wt):
            for c in range(4):
                for lane in range(64):
                    half, l32 = lane >> 5, lane & 31
                    row = (w * wt + i) * 32 + l32
                    at = row * KB + (((2 * c + half) ^ g.swz(row)) << 4)
                    assert along[at // 16] == (row, 2 * c + half)
                    pitch = g.pieces * 16
                    if esz == 4:                          # element e: contraction row 8 c + 4 half + e of column `row`
                        k0 = 8 * c + 4 * half
                        for e in range(4):
                            at = (k0 + e) * pitch + (((row >> 2) ^ g.kswz(k0)) << 4) + (row & 3) * 4
                            assert across[at // 16] == (k0 + e, row // 4) and at % 16 == row % 4 * 4
                        continue
                    trow = 8 * half + ((l32 & 15) >> 2)   # this lane's corner of the two transposing reads
                    piece = (w * 8 + i * 4 + (l32 >> 4) * 2 + ((l32 & 3) >> 1)) ^ g.kswz(trow)
                    for step in (0, 4):
                        at = (trow + c * 16) * pitch + piece * 16 + (l32 & 1) * 8 + step * pitch
                        col = (w * wt + i) * 32 + (l32 >> 4) * 16 + (l32 & 3) * 4  # four columns from here on
                        assert across[at // 16] == (trow + c * 16 + step, col * esz // 16) and at % 16 == col * esz % 16


def requests(g, layout, M, N, K, S, lda, ldb, idx):
    """(operand, base, size, offset checked, scalar offset, row in the operand, byte in the row, wanted) of every load."""
    esz = g.esz
    kbytes = K * esz
    a_kmajor = layout == "tn"
    nk = -(-K // g.krows) if a_kmajor else -(-kbytes // KB)
    a_rows = K if a_kmajor else S
    a_bytes, b_bytes = ((a_rows - 1) * lda + (M if a_kmajor else K)) * esz, ((S - 1) * ldb + N) * esz
    for m0 in range(0, M, g.rows):
        for n0 in range(0, N, g.rows):
            for kt in list(range(nk)) + [nk, nk + 3]:     # the loop asks for slabs past the end as well
                live = kt < nk
                left = kbytes - (kt * KB if live else 0)
                soff = kt * KB if live else 0
                for i in range(g.nld):
                    for t in {0, 1, 7, 8, 31, 64 * g.gw - 1}:
                        u = i * 64 * g.gw + t
                        kpos = ((t & 7) ^ g.swz(u // 8)) * 16
                        krow, kcol = u // g.pieces, ((u % g.pieces) ^ g.kswz(u // g.pieces)) * 16
                        k = kt * g.krows + krow
                        if a_kmajor:
                            off = kt * g.krows * lda * esz if live else 0
                            size = (K - 1) * lda * esz + (M - m0) * esz - off if live else 0
                            yield "A", m0 * esz + off, size, krow * lda * esz + kcol, 0, k, m0 * esz + kcol, live and k < K
                        else:
                            m = min(m0 + u // 8, M - 1)
                            row = idx[m] if layout == "nt" else m
                            yield ("A", 0, a_bytes if live else 0, row * lda * esz + kpos if kpos < left else (a_bytes if live else 0), soff, row,
                                   soff + kpos, live and soff + kpos < kbytes)
                        if layout == "nt":
                            size = (min(g.rows, N - n0) - 1) * ldb * esz + kbytes if live else 0
                            yield ("B", n0 * ldb * esz, size, (u // 8) * ldb * esz + kpos if kpos < left else size, soff, n0 + u // 8, soff + kpos,
                                   live and n0 + u // 8 < N and soff + kpos < kbytes)
                        elif layout == "nn":
                            off = kt * g.krows * ldb * esz if live else 0
                            size = (K - 1) * ldb * esz + (N - n0) * esz - off if live else 0
                            yield "B", n0 * esz + off, size, krow * ldb * esz + kcol, 0, k, n0 * esz + kcol, live and k < K
                        else:
                            row = idx[k] if k < K else 0
                            yield ("B", 0, b_bytes if live else 0, row * ldb * esz + n0 * esz + kcol if k < K else b_bytes, 0, row, n0 * esz + kcol,
                                   live and k < K)


@pytest.mark.parametrize("gw,esz,wt", SHAPES)
@pytest.mark.parametrize("layout,M,N,K,pad", [("nt", 130, 70, 72, 0), ("nt", 1, 1, 8, 8), ("nt", 65, 129, 200, 16), ("nn", 70, 136, 72, 0), ("nn", 129, 64, 200, 8),
                                              ("tn", 136, 72, 65, 0), ("tn", 64, 264, 131, 8), ("tn", 8, 8, 1, 0)])
def test_no_request_leaves_its_operand(gw, esz, wt, layout, M, N, K, pad):
    if layout == "nn" and esz == 4:
        pytest.skip("bf16 only")
    g = Geo(gw, esz, wt)
    S = (K if layout == "tn" else M) + 9
    idx = [(7 * r + 3) % S for r in range(K if layout == "tn" else M)]
    lda, ldb = (M if layout == "tn" else K) + pad, (K if layout == "nt" else N) + pad
    a_rows, b_rows = (K if layout == "tn" else S), {"nt": N, "nn": K, "tn": S}[layout]
    if layout == "nn":
        a_rows = S = M
    total = {"A": ((a_rows - 1) * lda + (M if layout == "tn" else K)) * esz, "B": ((b_rows - 1) * ldb + (K if layout == "nt" else N)) * esz}
    pitch = {"A": lda * esz, "B": ldb * esz}
    for op, base, size, voff, soff, row, byte, wanted in requests(g, layout, M, N, K, S, lda, ldb, idx):
        if voff + soff + 16 <= size:                      # the hardware lets it through
            assert 0 <= base + voff + soff <= total[op] - 16, (op, base, size, voff, soff)
        if wanted and byte + 16 <= (M if op == "A" and layout == "tn" else K if op == "A" or layout == "nt" else N) * esz:
            assert voff + soff + 16 <= size and base + voff + soff == row * pitch[op] + byte, (op, row, byte)
        if not wanted:
            assert voff >= size, (op, row, byte)          # arrives as zeros


def test_every_row_and_column_is_measured_once():
    """128 x 128 tiles, binary32: a wave follows the largest operand of its tile 0 of the rows and of the columns; wave (m, n) takes its
    row tiles in the order n, 1 - n and its column tiles in the order m, 1 - m."""
    waves = [(m, n) for m in range(2) for n in range(2)]
    assert sorted((m * 2 + (0 ^ n)) * 32 for m, n in waves) == sorted((n * 2 + (0 ^ m)) * 32 for m, n in waves) == [0, 32, 64, 96]
    sums = sorted(((m * 2 + (i ^ n)) * 32, (n * 2 + (j ^ m)) * 32) for m, n in waves for i in range(2) for j in range(2))
    assert sums == [(r, c) for r in range(0, 128, 32) for c in range(0, 128, 32)]


@pytest.mark.parametrize("nk", [1, 2, 3, 6])
def test_second_look_waits_for_its_slabs(nk):
    """128 x 128 tiles, binary32: the pass over all slabs that forms sums again keeps one slab on its way behind the one it reads; the
    indices of the kept rows (weight gradient) come two slabs ahead, into a ring of four entries."""
    stage, entry, on_the_way, reading = {}, {}, [], None

    def issue_tokens(kt):
        entry[kt % 4] = kt
        on_the_way.append(("tokens", kt))

    def load(kt):
        assert entry[kt % 4] == kt and ("tokens", kt) not in on_the_way
        assert reading is None or reading % 2 != kt % 2       # what is read at the same time lies in the other stage
        stage[kt % 2] = kt
        on_the_way.append(("slab", kt))
        issue_tokens(kt + 2)

    issue_tokens(0)
    issue_tokens(1)
    on_the_way.clear()                                        # waited for, then everyone's barrier
    load(0)
    for kt in range(nk):
        on_the_way.clear()
        reading = None                                        # everyone has read the slab before
        assert stage[kt % 2] == kt
        reading = kt
        load(kt + 1)
        assert stage[kt % 2] == kt and ("slab", kt) not in on_the_way
