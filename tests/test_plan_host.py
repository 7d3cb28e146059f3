"""Properties of the token-stream partition (section 4.4.3, "Layer 3": compute units balanced by token
count, long sequences split, short ones share a unit), checked on the CPU.  The functions under test
are the ones the kernels run (csrc/xattn_plan.h compiled for the host into the host test library);
only the wave-parallel sum and search of the device front end are replaced by plain loops there."""
import numpy as np
import pytest

import host_lib

GQA_COST, MLA_COST = 16, 192


def _cases():
    rng = np.random.RandomState(11)
    yield "tiny", [17, 64, 100, 256]
    yield "single token", [1]
    yield "all empty but one", [0, 0, 5, 0]
    yield "negative and zero lengths", [-3, 0, 40, -1, 0, 700, 0]
    yield "uniform 64", rng.randint(512, 4097, size=64)
    yield "long 16", rng.randint(16384, 32769, size=16)
    yield "lognormal 256", np.clip(np.rint(1024 * np.exp(1.2 * rng.randn(256))), 16, 65536).astype(np.int64)
    yield "one 65536-token sequence", [65536]
    yield "short ones around a long one", [3] * 50 + [65536] + [2] * 50
    yield "batch 4096 of short sequences", 1 + rng.randint(0, 40, size=4096)
    yield "batch 4096 with empties", rng.randint(0, 3, size=4096) * rng.randint(1, 30, size=4096)


CASES = list(_cases())
PARTITIONS = [(256, 64), (1, 16), (8, 16), (37, 48), (1024, 16), (65536, 16)]


def _all_segments(lens, n_pieces, min_piece, cost, skew=0):
    total, used = host_lib.plan(lens, n_pieces, min_piece, cost, skew)
    rows = []
    for p in range(used):
        for b, j0, j1, slot, whole in host_lib.piece_segments(lens, n_pieces, min_piece, cost, p, skew=skew):
            rows.append((p, b, j0, j1, slot, whole))
    return total, used, rows


@pytest.mark.parametrize("cost", [0, GQA_COST, MLA_COST])
@pytest.mark.parametrize("n_pieces,min_piece", PARTITIONS)
@pytest.mark.parametrize("name,lens", CASES, ids=[c[0] for c in CASES])
def test_pieces_tile_the_stream_and_balance(name, lens, n_pieces, min_piece, cost):
    lens = np.asarray(lens, np.int64)
    N = int(sum(L + cost for L in lens if L > 0))
    total, used = host_lib.plan(lens, n_pieces, min_piece, cost)
    assert total == N
    assert used == max(1, min(n_pieces, N // min_piece))
    bounds = host_lib.piece_bounds(lens, n_pieces, min_piece, cost)
    assert bounds[0] == 0 and bounds[-1] == N and len(bounds) == used + 1
    sizes = np.diff(bounds.astype(np.int64))
    if N > 0:
        assert np.all(sizes > 0), "an empty piece"
        assert np.all(bounds[:-1] % 16 == 0), "inner piece bounds are multiples of the 16-key block"
        assert np.all(np.abs(sizes - N / used) <= 16), "pieces differ from N / P by more than one block"
    # piece_of is the inverse of the bounds
    rng = np.random.RandomState(3)
    xs = set(int(x) for x in rng.randint(0, max(N, 1), size=64)) | set(int(b) for b in bounds[:-1]) | \
        set(int(b) - 1 for b in bounds[1:])
    for x in sorted(xs):
        if 0 <= x < N:
            assert host_lib.piece_of(lens, n_pieces, min_piece, cost, x) == int(np.searchsorted(bounds, x, side="right")) - 1


@pytest.mark.parametrize("cost,skew", [(0, 0), (GQA_COST, 0), (MLA_COST, 0), (GQA_COST, 32), (MLA_COST, 200)])
@pytest.mark.parametrize("n_pieces,min_piece", PARTITIONS[:5])
@pytest.mark.parametrize("name,lens", CASES, ids=[c[0] for c in CASES])
def test_every_token_is_in_exactly_one_segment(name, lens, n_pieces, min_piece, cost, skew):
    lens = np.asarray(lens, np.int64)
    B = len(lens)
    total, used, rows = _all_segments(lens, n_pieces, min_piece, cost, skew)
    bounds = host_lib.piece_bounds(lens, n_pieces, min_piece, cost, skew)
    covered = {b: [] for b in range(B)}
    slots = set()
    tokens_of_piece = np.zeros(used, np.int64)
    for p, b, j0, j1, slot, whole in rows:
        assert 0 <= b < B and 0 <= j0 < j1 <= lens[b], "an empty or out-of-range segment"
        assert slot == p + b and 0 <= slot < n_pieces + B
        assert slot not in slots, "two segments share a partial-result slot"
        slots.add(slot)
        assert bool(whole) == (j0 == 0 and j1 == lens[b])
        covered[b].append((j0, j1, p))
        tokens_of_piece[p] += j1 - j0
    for b in range(B):
        L = max(int(lens[b]), 0)
        segs = covered[b]                       # pieces are walked in stream order
        if L == 0:
            assert segs == []
            continue
        assert segs[0][0] == 0 and segs[-1][1] == L
        for (a0, a1, pa), (b0, b1, pb) in zip(segs, segs[1:]):
            assert a1 == b0 and pb == pa + 1, "segments of a sequence are contiguous, in consecutive pieces"
    # a piece never holds more tokens than positions
    assert np.all(tokens_of_piece <= np.diff(bounds.astype(np.int64)))
    assert int(tokens_of_piece.sum()) == int(lens[lens > 0].sum())


@pytest.mark.parametrize("cost,skew", [(GQA_COST, 0), (MLA_COST, 0), (GQA_COST, 32), (MLA_COST, 200)])
@pytest.mark.parametrize("n_pieces,min_piece", PARTITIONS[:5])
@pytest.mark.parametrize("name,lens", CASES, ids=[c[0] for c in CASES])
def test_segment_table_for_the_merge_equals_the_walk(name, lens, n_pieces, min_piece, cost, skew):
    lens = np.asarray(lens, np.int64)
    total, used, rows = _all_segments(lens, n_pieces, min_piece, cost, skew)
    meta = host_lib.meta(lens, n_pieces, min_piece, cost, skew)
    for b in range(len(lens)):
        mine = [r for r in rows if r[1] == b]
        first_slot, n_seg = int(meta[b, 0]), int(meta[b, 1])
        assert n_seg == len(mine)
        if mine:
            assert [r[4] for r in mine] == list(range(first_slot, first_slot + n_seg))
            assert (n_seg == 1) == bool(mine[0][5]), "exactly the unsplit sequences are finished by the decode kernel"


@pytest.mark.parametrize("skew", [1, 32, 200])
@pytest.mark.parametrize("n_pieces,min_piece", [(256, 64), (8, 16), (1024, 16), (65536, 16), (37, 48)])
@pytest.mark.parametrize("name,lens", CASES, ids=[c[0] for c in CASES])
def test_unequal_xcd_parts(name, lens, n_pieces, min_piece, skew):
    """With a skew the stream is cut into eight XCD parts, the even ones longer and the odd ones shorter
    by skew / 1000, each cut into equal pieces; the pieces still tile the stream and piece_of inverts
    the bounds.  Too few or too small pieces switch the skew off."""
    lens = np.asarray(lens, np.int64)
    N = int(sum(L + GQA_COST for L in lens if L > 0))
    total, used = host_lib.plan(lens, n_pieces, min_piece, GQA_COST, skew)
    assert total == N and used == max(1, min(n_pieces, N // min_piece))
    bounds = host_lib.piece_bounds(lens, n_pieces, min_piece, GQA_COST, skew).astype(np.int64)
    assert bounds[0] == 0 and bounds[-1] == N and len(bounds) == used + 1
    sizes = np.diff(bounds)
    if N == 0:
        return
    assert np.all(sizes > 0) and np.all(bounds[:-1] % 16 == 0)
    skewed = used % 8 == 0 and N // used >= 512
    if skewed:
        m = used // 8
        for x in range(8):
            want = N / used * (1 + skew / 1000.0 * (1 if x % 2 == 0 else -1))
            assert np.all(np.abs(sizes[x * m:(x + 1) * m] - want) <= 17), "XCD part %d" % x
            assert abs(bounds[x * m] - N * (x + (skew / 1000.0 if x % 2 else 0)) / 8) <= 9
    else:
        assert np.array_equal(bounds, host_lib.piece_bounds(lens, n_pieces, min_piece, GQA_COST, 0))
    rng = np.random.RandomState(4)
    xs = set(int(x) for x in rng.randint(0, N, size=64)) | set(int(b) for b in bounds[:-1]) | set(int(b) - 1 for b in bounds[1:])
    for x in sorted(xs):
        if 0 <= x < N:
            assert host_lib.piece_of(lens, n_pieces, min_piece, GQA_COST, x, skew) == int(np.searchsorted(bounds, x, side="right")) - 1


def test_stream_positions_up_to_the_32_bit_limit():
    """N just below 2^31 with the largest piece count: the 32-bit products of piece_bound do not wrap;
    beyond 2^31 - 1 the documented limit is reported, not wrapped."""
    lens = np.full(4096, 524287 - GQA_COST, np.int64)            # N = 4096 * 524287 = 2^31 - 4096
    N = 4096 * 524287
    for n_pieces, skew in ((256, 0), (65535, 0), (65536, 0), (256, 200), (65536, 32)):
        total, used = host_lib.plan(lens, n_pieces, 64, GQA_COST, skew)
        assert total == N and used == n_pieces
        bounds = host_lib.piece_bounds(lens, n_pieces, 64, GQA_COST, skew).astype(np.int64)
        assert bounds[0] == 0 and bounds[-1] == N
        sizes = np.diff(bounds)
        assert np.all(sizes > 0) and np.all(np.abs(sizes - N / used) <= 16 + N / used * skew / 1000.0)
        for x in (0, 1, N // 3, N - 1):
            assert host_lib.piece_of(lens, n_pieces, 64, GQA_COST, x, skew) == int(np.searchsorted(bounds, x, side="right")) - 1
    segs = host_lib.piece_segments(lens, 65536, 64, GQA_COST, 65535)
    assert segs[-1][0] == 4095 and segs[-1][2] == lens[-1]
    too_many = np.full(4096, 524288, np.int64)                   # N = 2^31 + ...: outside the limit
    assert host_lib.plan(too_many, 256, 64, GQA_COST) == (-1, -1)


# ----------------------------------------------------------------------------- short streams, the kernels' defaults
FEW_GQA, FEW_MLA = (256, 16), (32, 32)


def _short_streams():
    """Streams around the totals where the finer cut of short streams starts, is full and ends."""
    for total in (17, 31, 32, 33, 511, 512, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 16383, 16384, 16385, 40000):
        yield "one of %d" % total, [total]
    rng = np.random.RandomState(12)
    for n, hi in ((4, 300), (53, 100), (256, 16), (62, 84), (700, 5)):
        yield "%d of up to %d" % (n, hi), 1 + rng.randint(0, hi, size=n)
    yield "with empty ones", [0, 5, -2, 300, 0, 0, 17]


SHORT = list(_short_streams())


@pytest.mark.parametrize("cost,few,n_pieces,min_piece", [(GQA_COST, FEW_GQA, 256, 64), (GQA_COST, FEW_GQA, 1024, 64), (GQA_COST, FEW_GQA, 128, 64),
                                                         (GQA_COST, (37, 16), 256, 64), (MLA_COST, FEW_MLA, 256, 64), (96, FEW_MLA, 128, 64),
                                                         (MLA_COST, FEW_MLA, 256, 128), (MLA_COST, FEW_MLA, 128, 192)])
@pytest.mark.parametrize("name,lens", SHORT, ids=[c[0] for c in SHORT])
def test_short_streams_are_cut_finer(name, lens, cost, few, n_pieces, min_piece):
    lens = np.asarray(lens, np.int64)
    B, skew = len(lens), 32
    N = int(sum(L + cost for L in lens if L > 0))
    total, used = host_lib.plan(lens, n_pieces, min_piece, cost, skew, few)
    assert total == N
    assert used == max(1, min(n_pieces, max(N // min_piece, min(few[0], N // few[1]))))
    bounds = host_lib.piece_bounds(lens, n_pieces, min_piece, cost, skew, few).astype(np.int64)
    assert bounds[0] == 0 and bounds[-1] == N and len(bounds) == used + 1
    sizes = np.diff(bounds)
    assert np.all(sizes > 0) and np.all(bounds[:-1] % 16 == 0)
    for x in range(0, N, max(1, N // 997)):
        assert host_lib.piece_of(lens, n_pieces, min_piece, cost, x, skew, few) == int(np.searchsorted(bounds, x, side="right")) - 1
    # every key in one segment, slots unique, and the merge's table equal to the walk
    meta = host_lib.meta(lens, n_pieces, min_piece, cost, skew, few)
    seen = {b: [] for b in range(B)}
    slots = set()
    for p in range(used):
        for b, j0, j1, slot, whole in host_lib.piece_segments(lens, n_pieces, min_piece, cost, p, skew=skew, few=few):
            assert slot == p + b and slot < n_pieces + B and slot not in slots
            slots.add(slot)
            seen[b].append((j0, j1, slot, whole))
    for b in range(B):
        segs = seen[b]
        assert int(meta[b, 1]) == len(segs)
        if not segs:
            assert lens[b] <= 0
            continue
        assert segs[0][0] == 0 and segs[-1][1] == lens[b] and all(u[1] == v[0] for u, v in zip(segs, segs[1:]))
        assert [s[2] for s in segs] == list(range(int(meta[b, 0]), int(meta[b, 0]) + len(segs)))
        assert bool(segs[0][3]) == (len(segs) == 1)


@pytest.mark.parametrize("parts", [1, 2, 4, 8])
@pytest.mark.parametrize("n_pieces", [8, 37, 128, 256, 512, 1000, 2048])
def test_every_piece_and_row_has_one_workgroup_part(n_pieces, parts):
    """xattn_decode's map from workgroups to pieces and query rows, for every number of pieces that a stream may
    bring into use and 1 to 64 rows: each row of each piece in use is computed once, on the matrix path (16 or 32
    rows per wave; a tile per workgroup where enough of them are idle) and on the vector path (up to 8)."""
    used_counts = sorted({1, 2, 7, 8, 9, 15, 16, 17, n_pieces // 3 + 1, n_pieces // 2, n_pieces // 2 + 1, n_pieces - 1, n_pieces})
    narrow = wide = 0
    for used in used_counts:
        if not 1 <= used <= n_pieces:
            continue
        for rows in (1, 2, 3, 4, 8, 9, 15, 16, 17, 24, 31, 32, 33, 47, 48, 49, 63, 64):
            for rows_max in {8, 16 if rows <= 16 else 32}:
                total = 16 * used + 5
                got_rows, count = host_lib.decode_work(total, n_pieces, 64, GQA_COST, used, parts, rows, rows_max, few=(used, 16))
                assert np.all(count == 1), (used, rows, rows_max)
                assert got_rows == rows_max or (rows_max == 32 and got_rows == 16)
                if rows_max == 32:
                    narrow += got_rows == 16
                    wide += got_rows == 32
    assert n_pieces < 128 or (narrow and wide)          # both ways were taken


# ----------------------------------------------------------------------------- latent-KV weights
def _mla_streams():
    rng = np.random.RandomState(13)
    for n, lo, hi in ((78, 85, 342), (63, 172, 688), (128, 51, 410), (64, 1024, 8192), (30, 64, 256), (100, 64, 256), (16, 300, 1200),
                      (8, 2000, 9000), (5, 16, 8000), (300, 1, 40), (40, 500, 700)):
        yield "%d of %d to %d" % (n, lo, hi), rng.randint(lo, hi + 1, size=n)
    for n in (1, 129, 385, 1024, 2000, 5900, 6200, 24576, 30000, 50000):
        yield "one of %d" % n, [n]


MLA_STREAMS = list(_mla_streams())


def _segment_blocks(lens, n_pieces, min_piece, cost, few, keys):
    """Pieces in use, and the keys of every segment."""
    used = host_lib.plan(lens, n_pieces, min_piece, cost, 0, few)[1]
    segs = [host_lib.piece_segments(lens, n_pieces, min_piece, cost, p, few=few) for p in range(used)]
    return used, np.concatenate([s[:, 2] - s[:, 1] for s in segs]).astype(np.int64)


@pytest.mark.parametrize("rows", [33, 48, 64, 72, 128, 256, 384])
@pytest.mark.parametrize("name,lens", MLA_STREAMS, ids=[c[0] for c in MLA_STREAMS])
def test_mla_partition_keeps_the_share_of_exact_weights(name, lens, rows):
    """Keys past a segment's first exact blocks may enter the value product as one bf16 weight.  However the stream is
    cut, they are no more than with pieces of at least 64 positions, a segment cost of 192 and four such blocks, for
    which the error against the oracle was measured."""
    groups = (rows + 127) // 128
    n_pieces = 256 // groups // 8 * 8
    min_piece, cost, few, keys = host_lib.mla_cut(rows, len(lens))
    used, tokens = _segment_blocks(lens, n_pieces, min_piece, cost, few, keys)
    exact = host_lib.mla_exact_blocks(used, rows, n_pieces)
    _, bar_tokens = _segment_blocks(lens, n_pieces, 64, 192, (32, 32), keys)
    assert int(tokens.sum()) == int(bar_tokens.sum())
    assert np.maximum(tokens - exact * keys, 0).sum() <= np.maximum(bar_tokens - 4 * keys, 0).sum()
    if rows > 64 and used < n_pieces:           # the minimum cut the count: all blocks are exact
        assert tokens.max() <= exact * keys


@pytest.mark.parametrize("n_pieces", [1, 8, 37, 80, 128, 256, 1000])
def test_every_piece_and_tile_has_one_mla_workgroup(n_pieces):
    """The map from workgroups to pieces and tiles of 32 query rows, with short and with long pieces, for every number of
    pieces that a stream may bring into use: each tile of each piece in use is computed once."""
    seen = set()
    for used in sorted({1, 2, 7, 8, 9, 16, 17, n_pieces // 4, n_pieces // 2, n_pieces // 2 + 1, n_pieces - 1, n_pieces}):
        if not 1 <= used <= n_pieces:
            continue
        for rows in (33, 64, 65, 72, 96, 97, 128, 129, 192, 193, 261, 384, 4096):
            for positions in (64, 511, 512, 5000):           # per piece
                split, count = host_lib.mla_tile_work(positions * used, used, n_pieces, rows)
                assert np.all(count == 1), (used, rows, positions)
                seen.add((split, positions < 512))
                if split == 2:
                    assert positions < 512 and (used + 7) // 8 * ((rows + 63) // 64) <= (n_pieces + 7) // 8 * ((rows + 127) // 128)
    assert seen == {(1, True), (1, False), (2, True)}


@pytest.mark.parametrize("n,lo,hi,rows,split", [(8, 64, 256, 128, 2), (16, 20, 256, 72, 2), (30, 64, 256, 128, 2), (40, 64, 256, 128, 2),
                                                (40, 20, 256, 128, 2), (16, 64, 256, 256, 2), (4, 500, 3000, 128, 2), (29, 131, 262, 64, 2),
                                                (64, 1024, 8192, 128, 1), (64, 1024, 8192, 64, 1), (64, 64, 256, 256, 1)])
def test_short_mla_streams_halve_the_columns(n, lo, hi, rows, split):
    """Short sequences that leave workgroups idle: two waves per tile, above 64 query rows as well (with a tile per wave,
    calls of 16 to 40 sequences of 20 to 256 tokens spent most of their time at the start and end of a segment)."""
    rng = np.random.RandomState(14)
    lens = rng.randint(lo, hi + 1, size=n)
    n_pieces = 256 // ((rows + 127) // 128) // 8 * 8
    min_piece, cost, few, _ = host_lib.mla_cut(rows, n)
    total, used = host_lib.plan(lens, n_pieces, min_piece, cost, 0, few)
    assert host_lib.mla_tile_split(total, used, n_pieces, rows) == split
