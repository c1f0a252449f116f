"""The kernels' paths at the sizes where each can go wrong (edges of tiles,
remainders, smallest and largest of a range), bit-exact against the oracle."""
import numpy as np
import pytest

import datagen
import oracle
from tests.gpu_common import UINT64_MAX, as_u32, ids_tensor, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sel():
    if not torch.cuda.is_available():
        pytest.fail("gpu test run without a GPU")
    from paper_1806_08384_amd import sel as s
    return s


@pytest.fixture(scope="module")
def ctx(sel):
    c = sel.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def check(sel, ctx, dt, orc, tree):
    prog = ctx.program(dt, tree)
    want = orc.rowids(tree)
    assert ctx.count(dt, prog) == len(want), tree
    out = ids_tensor(len(want) + 1, torch)
    st, cnt = ctx.pushdown_rowids(dt, prog, UINT64_MAX, out)
    got = as_u32(out)
    assert st == sel.SEL_OK and cnt == len(want)
    np.testing.assert_array_equal(got[:cnt], want)
    assert got[cnt] == 0xDEADBEEF, "written past the count"


@pytest.mark.parametrize("tail", [1, 2, 3, 5, 255, 257, 1023, 2046, 2047])
@pytest.mark.parametrize("tiles", [0, 2, 13])
def test_partial_tile(sel, ctx, tiles, tail):
    """The table's last, partial tile: every column type (a dword of a narrow
    column may hold rows on both sides of the end), range, bitmap, hashed and
    plain sparse list and NULL tests, alone and after whole tiles, and
    selections of the last row alone."""
    n = 2048 * tiles + tail
    say(f"partial tile: {tiles} whole tiles + {tail} rows")
    rng = np.random.default_rng(n)
    t = datagen.random_table(rng, n, grid=False, null_rate=0.3)
    far = rng.integers(-2 ** 62, 2 ** 62, n)
    t.columns.append(datagen.Column("far", "i64", far))
    t.columns.append(datagen.Column("row", "i32", np.arange(n, dtype=np.int32)))
    dt = sel.device_table(ctx, t)
    orc = oracle.Oracle(t)
    some = tuple(int(v) for v in rng.choice(far, min(n, 40)))
    many = tuple(int(v) for v in rng.integers(-2 ** 62, 2 ** 62, 2000)) + some
    last = ("cmp", 5, "=", n - 1)
    trees = [last, ("not", last), ("in", 4, some), ("in", 4, many), ("or", ("in", 4, many), last)]
    for k in range(4):
        trees += [("between", k, -5, 9), ("in", k, (-3, 0, 7, 20)), ("isnull", k), ("not", ("cmp", k, "<", 0)),
                  ("codeset", k, 20, datagen.words_from_codes(range(0, 20, 3), 20))]
    trees.append(("and", *[("cmp", k, "<>", 1) for k in range(4)]))
    for tree in trees:
        check(sel, ctx, dt, orc, tree)
    # the batch kernels' partial tile
    pairs = [(dt, ctx.program(dt, tree)) for tree in trees]
    assert ctx.count_batch(pairs) == [orc.count(tree) for tree in trees]
    leaf = ("or", ("isunknown", ("cmp", 1, "<", 3)), ("in", 4, many))   # kept off the lookup tables
    assert ctx.count_batch([(dt, ctx.program(dt, leaf))]) == [orc.count(leaf)]


def test_results_are_each_calls_own(sel, ctx):
    """Counts come back through words that the kernels write to the host:
    calls of every kind in turn, on two contexts with streams of their own,
    each return their own result, an empty selection's 0 included."""
    n = 2048 * 9 + 700
    t = datagen.Table("own", n)
    t.columns.append(datagen.Column("row", "i32", np.arange(n, dtype=np.int32)))
    here = sel.device_table(ctx, t)
    other = sel.Context(0, stream=torch.cuda.Stream())
    there = sel.device_table(other, t)
    trees = [("cmp", 0, "<", k) for k in (0, 1, 2047, 2048, 2049, n - 1, n)]
    sides = []
    for c, dt in ((ctx, here), (other, there)):
        progs = [c.program(dt, tree) for tree in trees]
        sides.append((c, dt, progs, c.batch([(dt, p) for p in progs])))
    out = ids_tensor(n, torch)
    bits = torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda")
    want = [tree[3] for tree in trees]
    for k in range(3 * len(trees)):
        i = k % len(trees)
        for c, dt, progs, batch in sides:
            assert c.count(dt, progs[i]) == want[i]
            assert c.pushdown_rowids(dt, progs[i], UINT64_MAX, out) == (sel.SEL_OK, want[i])
            assert c.pushdown_keybitmap(dt, 0, 0, progs[-1 - i], bits, n) == (sel.SEL_OK, want[-1 - i])
            assert c.star_count(dt, [0], [bits], [n]) == want[-1 - i]
            assert c.count_batch([(dt, p) for p in progs]) == want
            assert batch.run() == want
    torch.cuda.synchronize()
    other.close()


@pytest.mark.parametrize("tiles", [1, 5, 3071, 3073, 4100])
@pytest.mark.parametrize("most", [1, 16, 17, 40, 2048])
def test_row_ids_by_density(sel, ctx, tiles, most):
    """Row ids where a tile has up to `most` TRUE rows, from none to all:
    four sparse tiles at once (up to 16 lanes with TRUE rows), a tile walked
    bit by bit and a dense one, in tables of one tile per scan wave and of
    more, with the partial tile at the end."""
    n = 2048 * tiles + 1111
    rng = np.random.default_rng(tiles + most)
    hit = np.zeros(n, dtype=np.int8)
    per = rng.integers(0, most + 1, tiles + 1)
    if most == 2048:
        per[::3] = 2048
    for t in range(tiles + 1):
        rows = min(2048, n - 2048 * t)
        lanes = 2048 * t + rng.choice(rows, min(int(per[t]), rows), replace=False)
        hit[lanes] = 1
        if t % 7 == 3 and per[t] > 3:      # several rows of one lane
            hit[2048 * t: 2048 * t + 4] = 1
    table = datagen.Table("density", n)
    table.columns.append(datagen.Column("hit", "i8", hit))
    dt = sel.device_table(ctx, table)
    want = np.flatnonzero(hit).astype(np.uint32)
    say(f"density: {tiles} tiles, up to {most}: {len(want)} ids")
    prog = ctx.program(dt, ("cmp", 0, "=", 1))
    for shape in (None, dict(block=64, grid=3), dict(block=128, tiles_per_step=4)):
        ctx.set_launch(**shape) if shape else ctx.set_launch()
        out = ids_tensor(len(want) + 1, torch)
        assert ctx.pushdown_rowids(dt, prog, UINT64_MAX, out) == (sel.SEL_OK, len(want))
        np.testing.assert_array_equal(as_u32(out)[:-1], want)
        assert as_u32(out)[-1] == 0xDEADBEEF
    ctx.set_launch()


@pytest.mark.parametrize("n", [1, 255, 511, 512, 513, 2048 * 37 + 1, (1 << 20) - 1, 1 << 20, (1 << 20) + 1])
def test_small_scan_sizes(sel, ctx, n):
    """Tables on both sides of the small scan's limit and of its quarter
    tiles, by the library's own launch and by a fixed one: counts, ids and key
    bitmaps, with a staged bitmap, a list too long for the small scan's LDS, a
    two-sided stack and NOTs and constants that fold into the leaf before."""
    rng = np.random.default_rng(n)
    t = datagen.random_table(rng, n, grid=False, null_rate=0.2)
    t.columns.append(datagen.Column("row", "i32", rng.permutation(n).astype(np.int32)))
    t.columns.append(datagen.Column("far", "i64", rng.integers(-2 ** 40, 2 ** 40, n)))
    t.columns.append(datagen.Column("code", "i32", rng.integers(0, 99_000, n).astype(np.int32), dict_card=99_000))
    dt = sel.device_table(ctx, t)
    orc = oracle.Oracle(t)
    half = datagen.words_from_codes(rng.choice(99_000, 40_000, replace=False), 99_000)
    few = datagen.words_from_codes(range(0, 60, 7), 60)
    many = tuple(int(v) for v in np.concatenate([rng.choice(t.columns[5].data, min(n, 900)),
                                                 rng.integers(-2 ** 40, 2 ** 40, 100)]))
    a, b, c, d = (("cmp", 0, ">", 2), ("between", 1, -9, 9), ("codeset", 6, 99_000, half), ("in", 5, many))
    trees = [a, c, d, ("codeset", 6, 60, few), ("and", ("not", a), c), ("or", ("not", ("not", d)), ("isnull", 2)),
             ("or", ("and", a, b), ("and", c, ("not", d))), ("and", ("true",), ("or", ("false",), b)),
             ("not", ("and", ("or", a, c), ("or", b, ("isunknown", ("cmp", 3, "<", 0))))),
             ("or", ("and", ("or", a, b), ("or", c, d)), ("and", ("or", b, ("notnull", 3)), ("or", ("not", a), d)))]
    say(f"small scan: {n} rows")
    if n > 100_000:
        trees = trees[4:6] + trees[9:]
    for shape in (None, dict(block=256, grid=40), dict(block=64, grid=7, cached=1)):
        ctx.set_launch(**shape) if shape else ctx.set_launch()
        for tree in trees:
            check(sel, ctx, dt, orc, tree)
            prog = ctx.program(dt, tree)
            for lo, bits in ((0, n), (n // 3, max(1, n // 2)))[:1 if n > 100_000 else 2]:
                bm = torch.full(((bits + 31) // 32,), -1, dtype=torch.int32, device="cuda")
                st, cnt = ctx.pushdown_keybitmap(dt, 4, lo, prog, bm, bits)
                ost, ocnt, words = orc.keybitmap(tree, 4, lo, bits)
                assert (st == sel.SEL_OK) == (ost == 0) and cnt == ocnt
                if st == sel.SEL_OK:
                    np.testing.assert_array_equal(as_u32(bm), words)
    ctx.set_launch()


@pytest.mark.parametrize("lo", [-37, 0, 5, 1000])
@pytest.mark.parametrize("width", [1, 31, 32, 33, 2046, 2047, 2048, 2049, 70_001])
@pytest.mark.parametrize("nprog", [3, 9, 20])
def test_batch_table_builds(sel, ctx, width, lo, nprog):
    """Lookup tables of both batch kernels at the edges of the builds' units
    (32 entries a thread, 64 or 2048 a unit) and entry widths: ranges, bitmaps
    of lists from any first value, NULLs, programs in conjunctive form and
    (IS UNKNOWN) not."""
    rng = np.random.default_rng(width + 3 * nprog + abs(lo))
    n = 6000
    data = rng.integers(lo - 3, lo + width + 3, n).astype(np.int32)
    t = datagen.Table("tab", n)
    t.columns.append(datagen.Column("x", "i32", data))
    valid = datagen.words_from_codes([i for i in range(n) if i % 7], n)
    t.columns.append(datagen.Column("y", "i32", data[::-1].copy(), valid))
    dt = sel.device_table(ctx, t)
    orc = oracle.Oracle(t)

    def leaf(col):
        a, b = sorted(int(v) for v in rng.integers(lo, lo + width, 2))
        if rng.random() < 0.4:
            return ("between", col, a, b)
        vals = set(int(v) for v in rng.integers(lo, lo + width, max(2, min(300, width // 3))))
        return ("in", col, tuple(vals | {a}))

    plain = [("and", leaf(0), ("or", leaf(1), leaf(0))) for _ in range(nprog)]
    other = [("and", leaf(0), leaf(0), leaf(0), ("not", ("isunknown", leaf(1)))) for _ in range(nprog)]
    for trees in (plain, other, plain + other):
        got = ctx.count_batch([(dt, ctx.program(dt, tree)) for tree in trees])
        assert got == [orc.count(tree) for tree in trees]


@pytest.mark.parametrize("rows", [4, 8])
@pytest.mark.parametrize("n", [1, 1023, 1025, 2048 * 25, 2048 * 49 + 1500])
def test_lookup_batch_columns(sel, ctx, n, rows):
    """The lookup-table kernel over passes of 1 to 16 columns of every type,
    with NULLs and without, windows and ranks, columns that only null tests
    read, and one-, two- and four-dword accumulators; both numbers of rows per
    lane, at the edges of quarter and half tiles and of the counters' reads."""
    rng = np.random.default_rng(n)
    t = datagen.random_table(rng, n, types=("i8", "i16", "i32", "i64") * 4, grid=False, null_rate=0.25)
    for k in (3, 7):       # wide values: ranks
        t.columns[k].data = rng.integers(-2 ** 61, 2 ** 61, n)
    dt = sel.device_table(ctx, t)
    orc = oracle.Oracle(t)

    def leaf(k):
        if k in (3, 7):
            return ("cmp", k, str(rng.choice(["<", ">="])), int(rng.integers(-2 ** 61, 2 ** 61)))
        r = rng.random()
        if r < 0.2:
            return ("isnull", k) if r < 0.1 else ("notnull", k)
        return ("between", k, int(rng.integers(-21, 5)), int(rng.integers(-4, 21)))

    def tree(cols, cross):
        parts = [leaf(int(c)) for c in cols]
        for _ in range(cross):
            a, b = (int(c) for c in rng.choice(cols, 2, replace=len(cols) < 2))
            parts.append(("or", leaf(a), ("not", leaf(b))))
        return parts[0] if len(parts) == 1 else ("and", *parts)

    ctx.set_launch(256, 0, rows_per_lane=rows)
    for ncols, nprog, cross in ((1, 2, 0), (2, 8, 1), (7, 16, 1), (9, 12, 2), (12, 9, 4), (16, 30, 1)):
        cols = rng.choice(16, ncols, replace=False)
        trees = [tree(rng.choice(cols, min(ncols, 1 + k % 4), replace=False), cross if ncols > 1 else 0)
                 for k in range(nprog)]
        got = ctx.count_batch([(dt, ctx.program(dt, x)) for x in trees])
        assert got == [orc.count(x) for x in trees], (ncols, nprog, cross)
    ctx.set_launch()


@pytest.mark.parametrize("nprog", [1, 8, 9, 15, 16, 17, 33])
def test_leaf_batch_words(sel, ctx, monkeypatch, nprog):
    """The leaf kernel over passes whose programs are all one TRUE word (read
    sixteen at a time) and passes where some are not, with each width of a
    lookup table's entries, leaves of conjunctions and of OR factors in one
    table, several leaves of one program in it, and a nullable column."""
    monkeypatch.setenv("SEL_BATCH_KERNEL", "leaf")
    rng = np.random.default_rng(nprog)
    n = 2048 * 27 + 700
    t = datagen.random_table(rng, n, types=("i8", "i16", "i32", "i32"), grid=False, null_rate=0.0)
    valid = datagen.words_from_codes([i for i in range(n) if i % 5], n)
    t.columns[1].valid = valid
    dt = sel.device_table(ctx, t)
    orc = oracle.Oracle(t)

    def leaf(k):
        if rng.random() < 0.5:
            return ("in", k, tuple(int(v) for v in rng.choice(np.arange(-20, 21), 9, replace=False)))
        return ("between", k, int(rng.integers(-21, 0)), int(rng.integers(0, 21)))

    one = [("and", *(leaf(k) for k in rng.permutation(4)), leaf(1), leaf(1)) for _ in range(nprog)]
    mixed = [("and", leaf(0), ("or", leaf(1), leaf(2)), leaf(1)) for _ in range(nprog)]
    for trees in (one, mixed, one + mixed + [("or", leaf(0), ("isunknown", leaf(1)))]):
        got = ctx.count_batch([(dt, ctx.program(dt, tree)) for tree in trees])
        assert got == [orc.count(tree) for tree in trees]


def test_timing_counts_every_batch_run(sel, ctx):
    """A batch run returns when its counts are there; read right after it, the
    timing holds that run: one launch, with a time."""
    n = 2048 * 40 + 9
    t = datagen.Table("timed", n)
    t.columns.append(datagen.Column("row", "i32", np.arange(n, dtype=np.int32)))
    dt = sel.device_table(ctx, t)
    pairs = [(dt, ctx.program(dt, ("cmp", 0, "<", k))) for k in (5, 700, n)]
    batch = ctx.batch(pairs)
    ctx.enable_timing(True)
    try:
        ctx.read_timing(reset=True)
        for k in range(60):
            assert batch.run() == [5, 700, n]
            ms, launches = ctx.read_timing(reset=True)
            assert launches[sel.K_BATCH] == 1 and ms[sel.K_BATCH] > 0, k
    finally:
        ctx.enable_timing(False)
        batch.destroy()


@pytest.mark.parametrize("tiles", [4095, 4096, 4097, 9000])
def test_row_ids_of_a_large_grid(sel, ctx, tiles):
    """Row ids where the caller's grid gives every tile a scan wave of its own,
    with few tiles and many: beyond 4096 tiles the counts go through their scan
    (each compaction wave adding up all counts before its own reads a number of
    them that grows with the square of the tiles)."""
    n = 2048 * tiles - 77
    rng = np.random.default_rng(tiles)
    hit = (rng.random(n) < 0.02).astype(np.int8)
    table = datagen.Table("grid", n)
    table.columns.append(datagen.Column("hit", "i8", hit))
    dt = sel.device_table(ctx, table)
    prog = ctx.program(dt, ("cmp", 0, "=", 1))
    want = np.flatnonzero(hit).astype(np.uint32)
    ctx.set_launch(block=256, grid=1 << 14)
    ctx.enable_timing(True)
    try:
        ctx.read_timing(reset=True)
        out = ids_tensor(len(want) + 1, torch)
        assert ctx.pushdown_rowids(dt, prog, UINT64_MAX, out) == (sel.SEL_OK, len(want))
        np.testing.assert_array_equal(as_u32(out)[:-1], want)
        assert as_u32(out)[-1] == 0xDEADBEEF
        _, launches = ctx.read_timing(reset=True)
        assert launches[sel.K_MASK] == 1 and launches[sel.K_COMPACT] == 1
        if tiles > 4096:
            assert launches[sel.K_SCAN] == 1
    finally:
        ctx.enable_timing(False)
        ctx.set_launch()


@pytest.mark.parametrize("stage", [0, 1])
@pytest.mark.parametrize("tail", [1, 63, 700, 2047])
def test_partial_tile_constants(sel, ctx, tail, stage):
    """A whole-tile scan's partial last tile with its constants staged in LDS
    and not: sorted lists short and long, hashed lists and bitmaps, on every
    column type, two of one list among them."""
    n = 2048 * 9 + tail
    rng = np.random.default_rng(tail)
    t = datagen.random_table(rng, n, grid=False, null_rate=0.2)
    t.columns.append(datagen.Column("far", "i64", rng.integers(-2 ** 62, 2 ** 62, n)))
    t.columns.append(datagen.Column("wide", "i32", rng.integers(-2 ** 31, 2 ** 31, n).astype(np.int32)))
    t.columns.append(datagen.Column("code", "i32", rng.integers(0, 9000, n).astype(np.int32), dict_card=9000))
    dt = sel.device_table(ctx, t)
    orc = oracle.Oracle(t)

    def some(k, m):
        x = t.columns[k].data
        lim = 2 ** 62 if k == 4 else 2 ** 31
        return tuple(int(v) for v in np.concatenate([x[-40:], rng.choice(x, 200), rng.integers(-lim, lim, m)]))

    codes = datagen.words_from_codes(rng.choice(9000, 3000, replace=False), 9000)
    trees = []
    for k in (4, 5):
        long, short = some(k, 1400), some(k, 30)
        trees += [("in", k, long), ("in", k, short), ("in", k, some(k, 7000)),
                  ("and", ("not", ("in", k, short)), ("in", k, long)), ("or", ("in", k, long), ("isnull", 1))]
    trees += [("codeset", 6, 9000, codes), ("and", ("codeset", 6, 9000, codes), ("in", 4, some(4, 1200)), ("cmp", 0, "<", 5))]
    trees += [("codeset", k, 20, datagen.words_from_codes(range(0, 20, 3), 20)) for k in range(4)]
    ctx.set_launch(block=256, grid=2, stage_words=stage)
    try:
        for tree in trees:
            check(sel, ctx, dt, orc, tree)
    finally:
        ctx.set_launch()


def test_partial_tile_is_no_slower(sel, ctx):
    """The partial last tile of a table does not hold up the scan: with a
    sorted list staged in LDS, rows short of a whole last tile cost no more
    than a quarter of the scan on top."""
    n = 2048 * 1500
    x = torch.randint(-2 ** 40, 2 ** 40, (n,), device="cuda", dtype=torch.int64)
    torch.cuda.synchronize()
    values = tuple(int(v) for v in np.random.default_rng(7).integers(-2 ** 40, 2 ** 40, 1500))
    best = []
    ctx.enable_timing(True)
    try:
        for rows in (n, n - 900):
            dt = ctx.table(rows, [("i64", 0, x.data_ptr(), None)], [x])
            prog = ctx.program(dt, ("in", 0, values))
            ms = []
            for _ in range(25):
                ctx.read_timing(reset=True)
                ctx.count(dt, prog)
                ms.append(ctx.read_timing(reset=True)[0][sel.K_COUNT])
            best.append(min(ms))
    finally:
        ctx.enable_timing(False)
    say("whole tiles", best[0], "partial last tile", best[1])
    assert best[1] < 1.25 * best[0]


@pytest.mark.parametrize("n", [1, 511, 2048 * 5 + 1501, (1 << 20) - 3, (1 << 20) + 2047, (1 << 21) + 1])
@pytest.mark.parametrize("key", ["i32", "i64"])
def test_key_bitmaps(sel, ctx, key, n):
    """Key bitmaps from both key types on both sides of the small scan's limit,
    at selections from one row of a tile to all, with keys in order and not,
    negative and (i64) beyond 32 bits, all in range and some out of it."""
    rng = np.random.default_rng(n)
    base = -(n // 2) if key == "i32" else int(rng.choice([-2 ** 40, 2 ** 33 + 5, -3]))
    t = datagen.Table("keys", n)
    dtype = np.int32 if key == "i32" else np.int64
    t.columns.append(datagen.Column("seq", key, (base + np.arange(n)).astype(dtype)))
    t.columns.append(datagen.Column("perm", key, (base + rng.permutation(n)).astype(dtype)))
    t.columns.append(datagen.Column("x", "i32", rng.integers(0, 10_000, n).astype(np.int32)))
    dt = sel.device_table(ctx, t)
    orc = oracle.Oracle(t)
    say(f"key bitmaps: {key} {n} rows")
    for shape in (None, dict(block=64, grid=11)):
        ctx.set_launch(**shape) if shape else ctx.set_launch()
        for below in (5, 300, 3000, 10_000):
            tree = ("cmp", 2, "<", below)
            prog = ctx.program(dt, tree)
            for col in (0, 1):
                for lo, bits in ((base, n), (base - 70, n + 100), (base + n // 3, max(1, n // 2))):
                    bm = torch.full(((bits + 31) // 32,), -1, dtype=torch.int32, device="cuda")
                    st, cnt = ctx.pushdown_keybitmap(dt, col, lo, prog, bm, bits)
                    ost, ocnt, words = orc.keybitmap(tree, col, lo, bits)
                    assert (st == sel.SEL_OK) == (ost == 0) and cnt == ocnt, (below, col, lo, bits)
                    if ost == 0:
                        np.testing.assert_array_equal(as_u32(bm), words)
    ctx.set_launch()


def test_selective_key_bitmap_reads_few_keys(sel, ctx):
    """A key bitmap of 0.5 % of a table's rows costs little more than their
    count: it does not read every key."""
    n = 100_000_000
    keys = torch.arange(n, device="cuda", dtype=torch.int64)
    x = torch.randint(0, 10_000, (n,), device="cuda", dtype=torch.int32)
    bits = torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    dt = ctx.table(n, [("i64", 0, keys.data_ptr(), None), ("i32", 0, x.data_ptr(), None)], [keys, x])
    prog = ctx.program(dt, ("cmp", 1, "<", 50))
    ctx.enable_timing(True)
    try:
        best = {}
        for kind, call in ((sel.K_COUNT, lambda: ctx.count(dt, prog)),
                           (sel.K_KEYBITMAP, lambda: ctx.pushdown_keybitmap(dt, 0, 0, prog, bits, n))):
            ms = []
            for _ in range(15):
                ctx.read_timing(reset=True)
                call()
                ms.append(ctx.read_timing(reset=True)[0][kind])
            best[kind] = min(ms)
    finally:
        ctx.enable_timing(False)
    say("count", best[sel.K_COUNT], "key bitmap", best[sel.K_KEYBITMAP])
    assert best[sel.K_KEYBITMAP] < 1.8 * best[sel.K_COUNT]


@pytest.mark.parametrize("tiles", [6, 4100])
@pytest.mark.parametrize("run", [2, 17, 32, 64, 700])
def test_row_ids_of_clustered_rows(sel, ctx, tiles, run):
    """Row ids where TRUE rows come in runs: words full and partly full, odd
    and even numbers of them in a compaction wave's tiles."""
    n = 2048 * tiles + 333
    rng = np.random.default_rng(run + tiles)
    for share in (0.01, 0.06, 0.12, 0.4):
        starts = np.flatnonzero(rng.random(n) < share / run)
        step = np.zeros(n + run + 1, dtype=np.int32)
        np.add.at(step, starts, 1)
        np.add.at(step, starts + run, -1)
        hit = (np.cumsum(step)[:n] > 0).astype(np.int8)
        table = datagen.Table("runs", n)
        table.columns.append(datagen.Column("hit", "i8", hit))
        dt = sel.device_table(ctx, table)
        want = np.flatnonzero(hit).astype(np.uint32)
        prog = ctx.program(dt, ("cmp", 0, "=", 1))
        for shape in (None, dict(block=64, grid=3)):
            ctx.set_launch(**shape) if shape else ctx.set_launch()
            out = ids_tensor(len(want) + 1, torch)
            assert ctx.pushdown_rowids(dt, prog, UINT64_MAX, out) == (sel.SEL_OK, len(want))
            np.testing.assert_array_equal(as_u32(out)[:-1], want)
            assert as_u32(out)[-1] == 0xDEADBEEF
    ctx.set_launch()


def test_short_runs_compact_like_long_ones(sel, ctx):
    """The same number of ids takes the compaction about the same time whether
    the rows come in runs of 700 or of 5000."""
    n = 200_000_000
    row = torch.arange(n, device="cuda")
    out = torch.empty(n // 8, dtype=torch.int32, device="cuda")
    best = {}
    ctx.enable_timing(True)
    try:
        for run in (5000, 700):
            hit = ((row // run) * 7919 % 1000 < 120).to(torch.int8)
            torch.cuda.synchronize()
            dt = ctx.table(n, [("i8", 0, hit.data_ptr(), None)], [hit])
            prog = ctx.program(dt, ("cmp", 0, "=", 1))
            ms = []
            for _ in range(15):
                ctx.read_timing(reset=True)
                st, cnt = ctx.pushdown_rowids(dt, prog, UINT64_MAX, out)
                assert st == sel.SEL_OK and abs(cnt - 0.12 * n) < 1e-3 * n
                ms.append(ctx.read_timing(reset=True)[0][sel.K_COMPACT])
            best[run] = min(ms)
    finally:
        ctx.enable_timing(False)
    say("compaction of runs", best)
    assert best[700] < 1.5 * best[5000]


@pytest.mark.parametrize("n", [2047, 2048, 2048 * 13 + 5, 2048 * 30])
def test_leaf_batch_sparse_lists(sel, ctx, monkeypatch, n):
    """Sparse IN lists in the leaf-major kernel: every column type, 1 to 700 values, first and last rows of steps
    and tiles among them, alone and under OR and NOT, NULLs."""
    monkeypatch.setenv("SEL_BATCH_KERNEL", "leaf")
    rng = np.random.default_rng(n)
    t = datagen.Table("lists", n)
    lims = {"i8": 2 ** 7, "i16": 2 ** 15, "i32": 2 ** 31, "i64": 2 ** 62}
    for ty, lim in lims.items():
        valid = datagen.words_from_codes([i for i in range(n) if i % 5], n) if ty in ("i16", "i64") else None
        t.columns.append(datagen.Column(ty, ty, rng.integers(-lim, lim, n).astype("int" + ty[1:]), valid))
    t.columns.append(datagen.Column("f", "i8", rng.integers(-9, 9, n).astype(np.int8),
                                    datagen.words_from_codes([i for i in range(n) if i % 3], n)))
    dt = sel.device_table(ctx, t)
    orc = oracle.Oracle(t)
    trees = []
    for k, lim in enumerate(lims.values()):
        x = t.columns[k].data
        edges = x[[i for i in (0, 3, 4, 255, 256, 259, 1023, 2046, 2047, n - 1) if i < n]]
        for m in (0, 2, 30, 690):
            vals = tuple(int(v) for v in np.concatenate([edges, rng.integers(-lim, lim, m)]))[: max(1, m + 10)]
            known = ("not", ("isunknown", ("cmp", 4, "<", 3)))
            trees += [("and", known, ("in", k, vals)), ("or", ("isunknown", ("cmp", 4, ">", 5)), ("not", ("in", k, vals)))]
    for j in range(0, len(trees), 8):
        got = ctx.count_batch([(dt, ctx.program(dt, x)) for x in trees[j:j + 8]])
        assert got == [orc.count(x) for x in trees[j:j + 8]], j


def test_leaf_batch_lists_against_counts(sel, ctx, monkeypatch):
    """Six sparse int64 lists in one leaf-major batch take less than 2.6 times
    the counts of the lists one by one."""
    n = 60_000_000
    x = torch.randint(-2 ** 40, 2 ** 40, (n,), device="cuda", dtype=torch.int64)
    torch.cuda.synchronize()
    dt = ctx.table(n, [("i64", 0, x.data_ptr(), None)], [x])
    rng = np.random.default_rng(5)
    monkeypatch.setenv("SEL_BATCH_KERNEL", "leaf")
    lists = [("in", 0, tuple(int(v) for v in rng.integers(-2 ** 40, 2 ** 40, 3))) for _ in range(6)]
    one = [ctx.program(dt, t) for t in lists]
    batch = ctx.batch([(dt, p) for p in one])
    want = [ctx.count(dt, p) for p in one]
    ctx.enable_timing(True)
    try:
        best = {sel.K_COUNT: [], sel.K_BATCH: []}
        for _ in range(12):
            ctx.read_timing(reset=True)
            assert [ctx.count(dt, p) for p in one] == want
            assert batch.run() == want
            ms, launches = ctx.read_timing(reset=True)
            assert launches[sel.K_COUNT] == 6 and launches[sel.K_BATCH] == 1
            for kind in best:
                best[kind].append(ms[kind])
    finally:
        ctx.enable_timing(False)
        batch.destroy()
    count, together = min(best[sel.K_COUNT]), min(best[sel.K_BATCH])
    say("counts", count, "batch", together)
    assert together < 2.6 * count
