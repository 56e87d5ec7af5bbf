"""Which kernels a call launches, and what it does under capture and when memory runs out: the library's host code on a HIP
runtime without a device (tests/stub_library.py)."""
import pytest

import stub_library


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    return stub_library.link(str(tmp_path_factory.mktemp("stub")))


@pytest.fixture
def ctx(library):
    c = stub_library.StubContext(library)
    yield c
    c.close()


def test_captured_small_epochs_clear_their_own_sums(library):
    """A replay finds what the replay before it has left, not what the host counted on: a captured small epoch starts by
    clearing its sums.  Eager ones need that only where the call before has not cleared as much."""
    ctx = stub_library.StubContext(library, stream=0x1000)
    try:
        small = ["small_kernel<2,true>", "small_update_kernel"]
        assert ctx.epoch(5000, 100, 8) == (0, ["fill_zero_kernel"] + small)
        assert ctx.epoch(5000, 100, 8) == (0, small)
        ctx.capturing(True)
        for _ in range(2):
            assert ctx.epoch(5000, 100, 8) == (0, ["fill_zero_kernel"] + small)
        ctx.capturing(False)
        assert ctx.epoch(5000, 100, 8) == (0, small)
        assert ctx.epoch(5000, 49, 8) == (0, small)                                   # a smaller map
        assert ctx.epoch(5000, 100, 8) == (0, ["fill_zero_kernel"] + small)           # a larger one
        assert ctx.epoch(5000, 100, 8) == (0, small)
    finally:
        ctx.close()


# (K, D, most rows of a look-up in one kernel, that kernel).  lookup_kernel: full rounds of 8 rows x 256 units x workgroups on
# a unit; small_kernel: a power of two of the rows, or (few nodes, or fewer than four features) m K D <= 4e8.
@pytest.mark.parametrize("K,D,rows,kernel", [
    (64, 50, 2 * 3 * 2048, "lookup_kernel<8>"), (128, 33, 2 * 3 * 2048, "lookup_kernel<8>"), (400, 50, 2 * 2 * 2048, "lookup_kernel<8>"),
    (512, 50, 2 * 2048, "lookup_kernel<8>"), (1024, 50, 2048, "lookup_kernel<8>"), (1024, 64, 2048, "lookup_kernel<8>"),
    (4096, 64, 1525, "lookup_kernel<8>"), (20000, 64, 312, "lookup_kernel<4>"), (1500, 40, 2 * 2048, "lookup_kernel<8>"),
    (2048, 16, 2 * 2048, "lookup_kernel<8>"), (4096, 8, 3 * 2048, "lookup_kernel<8>"), (9000, 3, 14814, "lookup_kernel<8>"),
    (100, 8, 500_000, "small_kernel<2,false>"), (128, 16, 195_312, "small_kernel<4,false>"), (16, 4, 6_250_000, "small_kernel<1,false>"),
    (129, 16, 262_143, "small_kernel<4,false>"), (400, 32, 32_767, "small_kernel<8,false>"), (1024, 5, 65_535, "small_kernel<2,false>"),
    (4096, 4, 32_767, "small_kernel<1,false>"), (1024, 2, 195_312, "small_kernel<1,false>"),
])
def test_look_ups_on_both_sides_of_their_line(ctx, K, D, rows, kernel):
    assert ctx.bmu(rows, K, D) == (0, [kernel])
    assert ctx.launches[0][5] < 160 * 1024 - 1024            # LDS of a unit, beside the kernel's own few hundred bytes
    assert ctx.bmu(rows, K, D, qe=True) == (0, [kernel, "small_qe_kernel"])
    rc, names = ctx.bmu(rows + 1, K, D)
    assert rc == 0 and not any(n.startswith(("lookup", "small")) for n in names) and len(names) >= 4
    # a profile, and the float32 search, are of the general path
    for switch, on, off in (("som_profile", 1, 0), ("som_set_search", 1, 0)):
        ctx.switch(switch, on)
        rc, names = ctx.bmu(1000, K, D)
        assert rc == 0 and not any(n.startswith(("lookup", "small")) for n in names)
        ctx.switch(switch, off)
    rc, names = ctx.bmu(1000, K, 65)
    assert rc == 0 and "bmu_wide_split_kernel" in names      # rows of more than 64 features


def test_look_ups_take_no_more_threads_than_nodes_are_worth(ctx):
    """A workgroup's time goes with ceil(K / 512) and not with K: tens of thousands of rows on a map of few nodes are not a
    small look-up (12,500 workgroups at 100,000 rows of 50 features on 80 nodes)."""
    for K in (16, 64, 80, 128, 256, 400):
        rc, names = ctx.bmu(20_000, K, 50)
        assert rc == 0 and any(n.startswith("bmu_split_kernel") for n in names), (K, names)


SORT = ["sort_hist_kernel", "sort_columns_kernel", "sort_starts_kernel", "sort_scatter_kernel", "sort_sums_kernel", "sort_finish_kernel"]
STABLE = ["stable_hist_kernel", "sort_columns_kernel", "sort_starts_kernel", "stable_scatter_kernel", "sort_sums_kernel", "sort_finish_kernel"]
SLABS = ["accumulate_f64_kernel", "accumulate_f64_reduce_kernel"]
MFMA = ["accumulate_mfma_kernel", "accumulate_mfma_reduce_kernel"]
FLOAT32 = ["accumulate_kernel", "accumulate_reduce_kernel"]


def plain(result):
    rc, names = result
    return rc, [n.split("<")[0] for n in names]


@pytest.mark.parametrize("m,K,D,kernels", [
    (1_000_000, 1024, 50, SLABS), (749_999, 4096, 50, SLABS), (750_000, 4096, 50, SORT), (1_000_000, 3136, 50, SLABS),
    (1_000_000, 6401, 40, SLABS), (1_000_000, 6400, 40, SORT), (5_000_000, 16384, 16, SLABS), (100, 16384, 50, SORT),
    (255, 16, 64, 2 * SLABS), (256, 16, 64, SORT), (1023, 1024, 126, 2 * SLABS), (1024, 1024, 126, SORT), (10, 1024, 127, SORT),
    (799_999, 1024, 96, SORT), (800_000, 1024, 65, 2 * SLABS), (800_000, 1024, 96, 2 * SLABS), (800_000, 1024, 64, SORT),
    (800_000, 1024, 97, SORT), (499_999, 4096, 64, 2 * SLABS), (500_000, 4096, 64, SORT), (800_000, 4096, 72, SORT),
    (10, 16, 2000, SORT), (1000, 16385, 200, FLOAT32), (1000, 16385, 16, SLABS), (1000, 16385, 63, FLOAT32),
])
def test_accumulation_routes(ctx, m, K, D, kernels):
    for zero_first in (True, False):
        assert plain(ctx.accumulate(m, K, D, zero_first)) == (0, kernels)


def test_accumulation_of_rows_far_apart_keeps_float64_sums(ctx):
    """The slab kernel's row offsets hold strides below 2^22 floats; beyond them the sort serves every call that it can."""
    for m, K, D in ((100, 1024, 100), (1_000_000, 1024, 72), (1000, 4096, 50), (1000, 16, 8)):
        assert plain(ctx.accumulate(m, K, D, ldx=(1 << 22) - 1))[1][0] == SLABS[0]
        assert plain(ctx.accumulate(m, K, D, ldx=1 << 22)) == (0, SORT)


def test_accumulation_without_memory_for_the_sort(ctx):
    """The sort's workspace goes with the samples; the kernels that served such calls before it need less, and do again."""
    m, K, D = 20_000_000, 100, 200
    ctx.limit(64 << 20)                                          # the sort asks for 80 MB and more here
    assert plain(ctx.accumulate(m, K, D)) == (0, 4 * SLABS)
    # a fixed order stays a fixed order: the MFMA accumulators where they apply, an error elsewhere
    ctx.switch("som_set_reproducible", 1)
    assert plain(ctx.accumulate(m, K, D)) == (0, 4 * MFMA)
    assert plain(ctx.accumulate(m, 4096, D)) == (-2, []) and "accumulation workspace" in ctx.error()
    ctx.limit()
    assert plain(ctx.accumulate(m, K, D)) == (0, STABLE)
    assert plain(ctx.accumulate(m, 4096, D)) == (0, STABLE)
    ctx.switch("som_set_reproducible", 0)
    assert plain(ctx.accumulate(m, K, D)) == (0, SORT)
    # nothing at all: an error, and the context works afterwards
    ctx.limit(1 << 10)
    assert plain(ctx.accumulate(2 * m, K, D))[0] == -2
    ctx.limit()
    assert plain(ctx.accumulate(2 * m, K, D)) == (0, SORT)


@pytest.mark.parametrize("kernel", ["small_kernel", "small_update_kernel"])
def test_a_small_epoch_that_failed_leaves_nothing_behind(ctx, kernel):
    """Neither launch of a failed epoch is counted on: the next one clears its sums itself."""
    small = ["small_kernel<2,true>", "small_update_kernel"]
    assert ctx.epoch(5000, 100, 8) == (0, ["fill_zero_kernel"] + small)
    ctx.fail(kernel)
    rc, names = ctx.epoch(5000, 100, 8)
    assert rc == -3 and "small-map" in ctx.error()
    ctx.fail()
    assert ctx.epoch(5000, 100, 8) == (0, ["fill_zero_kernel"] + small)
    assert ctx.epoch(5000, 100, 8) == (0, small)


@pytest.mark.parametrize("kernel", ["bmu_split_prep_kernel", "bmu_split_kernel", "bmu_list_kernel"])
def test_a_search_that_failed_before_its_list_leaves_no_maxima_behind(ctx, kernel):
    """The maxima that the preparation finds are zero again once the list kernel has run; a call that did not get there makes
    the next one clear them.  Another search in between does not touch them."""
    rc, usual = ctx.bmu(100_000, 300, 50)
    assert rc == 0 and usual[0] == "fill_zero_kernel" and usual[1] == "bmu_split_prep_kernel"
    rc, again = ctx.bmu(100_000, 300, 50)
    assert rc == 0 and again == usual[1:]
    ctx.fail(kernel)
    assert ctx.bmu(100_000, 300, 50)[0] == -3
    ctx.fail()
    assert ctx.bmu(100_000, 300, 50) == (0, usual)
    assert ctx.bmu(100, 50, 3)[0] == 0                                    # (a small look-up, and the float32 search)
    ctx.switch("som_set_search", 1)
    assert ctx.bmu(5000, 200, 50)[0] == 0
    ctx.switch("som_set_search", 0)
    assert ctx.bmu(100_000, 300, 50) == (0, again)
    assert ctx.bmu(100_000, 3000, 50)[1][:2] == ["fill_zero_kernel", "bmu_split_prep_kernel"]     # a new allocation


# small epochs: without statistics, in the default mode, up to 32 features, 512 nodes, m K D = 3e8, W and the sums in LDS
@pytest.mark.parametrize("m,K,D,small", [
    (375_000, 100, 8, True), (375_001, 100, 8, False), (4000, 200, 32, True), (4000, 200, 33, False), (3000, 512, 8, True),
    (3000, 513, 8, False), (3000, 334, 32, True), (3000, 335, 32, False), (10, 1, 1, True)])
def test_small_epochs_on_both_sides_of_their_limits(ctx, m, K, D, small):
    rc, names = ctx.epoch(m, K, D)
    assert rc == 0 and (names[-1] == "small_update_kernel") == small, names
    assert all(lds <= 160 * 1024 - 1024 for *_, lds in ctx.launches)
    for switch in ("som_profile", "som_set_search", "som_set_reproducible"):
        ctx.switch(switch, 1)
        rc, names = ctx.epoch(m, K, D)
        ctx.switch(switch, 0)
        assert rc == 0 and "small_update_kernel" not in names


def test_dynamic_lds_is_raised_on_every_device(library):
    """The limit on a kernel's dynamic LDS belongs to the device: a second one needs it raised as the first did."""
    contexts = [stub_library.StubContext(library, device=d) for d in (0, 1)]
    try:
        for ctx in contexts:
            for search in (0, 1):
                ctx.switch("som_set_search", search)
                for D in (8, 16, 17, 24, 32, 33, 40, 50, 55, 64, 100, 130, 200):
                    for K in (64, 400, 1024):
                        assert ctx.bmu(200_000, K, D)[0] == 0 and ctx.bmu(500, K, D)[0] == 0, (search, K, D, ctx.error())
                        assert ctx.epoch(3000, K, D)[0] == 0, (search, K, D, ctx.error())
            for fixed in (0, 1):
                ctx.switch("som_set_reproducible", fixed)
                for K, D in ((300, 3), (1024, 3), (2000, 31), (8000, 100), (12_000, 70), (18_000, 40), (6000, 63)):
                    for m in (100_000, 10_000_000):
                        assert ctx.accumulate(m, K, D)[0] == 0, (fixed, m, K, D, ctx.error())
    finally:
        for ctx in contexts:
            ctx.close()


def test_wide_rows_on_both_sides_of_their_lines(ctx):
    """Rows of 65 to 256 features are held in registers; wider ones are cut beforehand on maps of more than 320 nodes, or of more than 512 where
    the rows are many and fill the tile's rounds (the more of them the more nodes there are, and the less chunks of 32 features save)."""
    for m, K, D, cut in ((1000, 321, 256, False), (1000, 320, 257, False), (1000, 321, 257, True), (1000, 1024, 2000, True), (1000, 70000, 300, True),
                         (131_072, 321, 257, False), (131_072, 448, 600, False), (131_072, 449, 600, True), (131_073, 448, 600, True), (126_000, 448, 600, True),
                         (250_000, 400, 300, False), (262_144, 512, 300, False), (262_144, 513, 300, True), (250_000, 512, 300, True),
                         (250_000, 449, 320, True), (324_149, 500, 270, False)):
        rc, names = ctx.bmu(m, K, D)
        assert rc == 0 and names.count("bmu_cut_samples_kernel") == cut and ("bmu_wide_split_kernel" in names) != cut, (K, D, names)


# workgroups: whole rounds of sample tiles (counted by eights) times their pieces, and the tiles left over times theirs
@pytest.mark.parametrize("m,K,groups", [
    (100_000, 1024, 384 * 4 + 8 * 16), (50_497, 800, 192 * 4 + 8 * 13), (100_000, 1600, 384 * 4 + 8 * 13), (10_000, 600, 40 * 5),
    (140_000, 600, 512 * 3 + 40 * 3),                             # (a short last piece behind whole rounds of three)
    (65_536, 1024, 256 * 4), (10_000, 1024, 40 * 4), (10_618, 729, 48 * 3), (1000, 4100, 8 * 9)])
def test_the_last_round_of_rows_cut_beforehand_goes_in_smaller_pieces(ctx, m, K, groups):
    rc, names = ctx.bmu(m, K, 600)
    assert rc == 0 and [w[1] for w in ctx.launches if w[0] == "bmu_cut_split_kernel"] == [groups]


def test_smaller_pieces_take_memory_for_their_own_rows_only(ctx):
    """Sixteen pieces of the last tiles don't make every row's results sixteen: 300,000 rows on 1024 nodes and the whole rounds among them."""
    whole, more = 65_536 * 4, 65_536 * 4 + 256 * 4
    assert ctx.bmu(whole, 1024, 300)[0] == 0 and [w[1] for w in ctx.launches if w[0] == "bmu_cut_split_kernel"] == [whole // 256 * 4]
    ctx.lib.stub_peak_reset()
    assert ctx.bmu(more, 1024, 300)[0] == 0 and [w[1] for w in ctx.launches if w[0] == "bmu_cut_split_kernel"] == [whole // 256 * 4 + 8 * 16]
    per_row = 5 * 228 + 16 + 32                                   # parts, scales, norm, record; and 32 bytes a result
    assert ctx.lib.stub_peak() <= more * (per_row + 4 * 32) + 1024 * 12 * 32 + 4096


def test_rows_cut_beforehand_go_in_passes_that_memory_holds(ctx):
    """The parts of a pass take at most a gigabyte, and where an allocation fails, half as many rows, down to a tile's."""
    passes = lambda m, K, D: ctx.bmu(m, K, D)[1].count("bmu_cut_samples_kernel")
    ctx.limit(10 << 20)                                          # the preparation takes 7.6 MB
    rc, names = ctx.bmu(3000, 400, 2000)
    assert rc == 0 and names.count("bmu_cut_samples_kernel") > 1
    ctx.limit(64 << 20)
    assert passes(100_000, 400, 2000) in range(12, 27)
    ctx.limit()
    per = (1 << 30) // (32 * 228) // 256 * 256                   # 32 chunks of 64 features, a row's 224 bytes and a scale each
    assert passes(per, 400, 2000) == 1 and passes(per + 1, 400, 2000) == 2


# bytes a row: list, cut and mark; two words of pair ids on small maps and four on large ones, for rows of up to 64 features only
@pytest.mark.parametrize("K,D,search,per_row", [(400, 50, 0, 20), (1023, 50, 0, 20), (1024, 50, 0, 28), (3000, 20, 0, 28), (400, 50, 1, 12 + 32), (1024, 3, 0, 12 + 32)])
def test_bytes_of_the_lists(library, K, D, search, per_row):
    ctx = stub_library.StubContext(library)
    try:
        ctx.switch("som_set_search", search)
        assert ctx.bmu(1000, K, D)[0] == 0
        m, before = 4_000_000, ctx.in_use()
        assert ctx.bmu(m, K, D)[0] == 0
        assert per_row * (m - 100_000) <= ctx.in_use() - before <= per_row * m + 4 * K * (4 * D + 1000)
    finally:
        ctx.close()


@pytest.mark.parametrize("K,D,search,kernel,per_row", [(400, 50, 0, "bmu_split_kernel", 12), (1024, 50, 0, "bmu_split_kernel", 16),
                                                       (300, 50, 1, "bmu_kernel", 44)])
@pytest.mark.parametrize("passes", [1, 2, 4])
def test_searches_without_memory_for_their_lists_go_in_passes(library, K, D, search, kernel, per_row, passes):
    """Half as many rows where the largest allocation of a pass fails, and again; an error where nothing is left."""
    ctx = stub_library.StubContext(library)
    try:
        ctx.switch("som_set_search", search)
        m = 1_000_000
        ctx.limit(m // passes * per_row + (1 << 16))
        rc, names = ctx.bmu(m, K, D)
        assert rc == 0 and sum(n.split("<")[0] == kernel for n in names) == passes, names
        ctx.limit(1 << 10)
        assert ctx.bmu(4 * m, 9 * K, D)[0] == -2
        ctx.limit()
        assert ctx.bmu(4 * m, K, D)[0] == 0
    finally:
        ctx.close()


@pytest.mark.parametrize("m,K,D,kernel,limit", [(100_000, 400, 2000, "bmu_cut_samples_kernel", 64 << 20), (1_000_000, 1024, 50, "bmu_split_kernel", 5 << 20)])
def test_passes_that_memory_held_are_kept(library, m, K, D, kernel, limit):
    """The same call again starts with the rows that memory held: nothing is allocated and nothing given back.  With more memory it tries
    again, and what fails then is kept in turn; another call is not touched."""
    ctx = stub_library.StubContext(library)
    passes = lambda *call: [n.split("<")[0] for n in ctx.bmu(*call)[1]].count(kernel)
    moved = lambda: (ctx.lib.stub_allocated(), ctx.lib.stub_freed())
    try:
        ctx.lib.stub_taken(1 << 30)                               # (somebody else's)
        ctx.limit(limit)
        few = passes(m, K, D)
        assert few > 1
        before = moved()
        for _ in range(3):
            assert passes(m, K, D) == few and moved() == before
        assert passes(m // 50, K, D) == 1 and passes(m, K, D) == few and moved() == before
        ctx.lib.stub_taken(1 << 20)                               # more is left, but allocations fail as before
        assert passes(m, K, D) == few and moved()[1] > before[1]
        before = moved()
        assert passes(m, K, D) == few and moved() == before
        ctx.limit()
        assert passes(m, K, D) == few and moved() == before
        ctx.lib.stub_taken(0)
        assert passes(m, K, D) == 1
        before = moved()
        ctx.limit(limit)
        assert passes(m, K, D) == 1 and moved() == before
        ctx.limit(1 << 10)                                        # a call that fails altogether is not kept: the next one asks for all rows
        assert ctx.bmu(m * 13 // 10, K, D)[0] == -2
        ctx.limit()
        assert passes(m * 13 // 10, K, D) == 1
    finally:
        ctx.lib.stub_taken(0)
        ctx.limit()
        ctx.close()


def test_the_first_call_knows_the_units_of_its_device(library):
    """131,072 rows fill the tile's rounds on 128 units and not on 256: the first call of a context takes the form that later ones take, and
    sizes their workspaces."""
    for units, cut in ((128, 0), (256, 1)):
        library_units = stub_library.C.CDLL(library).stub_units
        library_units(units)
        ctx = stub_library.StubContext(library)
        try:
            first = ctx.bmu(131_072, 400, 300)
            held = ctx.lib.stub_allocated()
            assert first[0] == 0 and first[1].count("bmu_cut_samples_kernel") == cut
            assert ctx.bmu(131_072, 400, 300) == first and ctx.lib.stub_allocated() == held
        finally:
            library_units(256)
            ctx.close()
