"""The rules by which launches are cut (csrc/split_plan.hpp, score_tile.hpp, stats_bulk.hpp, step_rule.hpp, dense_plan.hpp:
host arithmetic), compiled here without HIP."""
import ctypes as C
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
MORE_BYTES = 256 << 10  # how much longer than a chunk of most_splits a chunk may be


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rules") / "launch_rules.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-ftrapv", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "c_abi", "launch_rules.cpp")], check=True)
    c = C.CDLL(so)

    class Lib:
        @staticmethod
        def most(rows, length):
            out = (C.c_int * 3)()
            c.most(rows, length, out)
            return tuple(out)

        @staticmethod
        def plan(batch, heads, length, max_pages, page_bytes, slow=0):
            out = (C.c_int * 3)()
            c.plan(batch, heads, length, max_pages, page_bytes, slow, out)
            return tuple(out)

        @staticmethod
        def tile(batch, heads, head_dim, max_pages, min_pages, max_tile=256):
            return c.tile(batch, heads, head_dim, max_pages, min_pages, max_tile)

        @staticmethod
        def bulk(mb, head_dim, page_size, key_bytes, bf16_means):
            return bool(c.bulk(C.c_longlong(mb << 20), head_dim, page_size, key_bytes, int(bf16_means)))

        @staticmethod
        def fuses(batch, heads, max_pages, top_k, page_bytes=8192):
            return bool(c.fuses(batch, heads, max_pages, top_k, page_bytes))

        @staticmethod
        def fuses_of(batch, heads, max_pages, top_k, page_size=16, head_dim=128, bf16=True):
            return bool(c.fuses_of(batch, heads, max_pages, top_k, page_size, head_dim, int(bf16)))

        @staticmethod
        def score_grid(cut, tiles, batch, heads, n_bytes, group, fitted=False):
            out = (C.c_int * 4)()
            c.score_grid(int(cut), tiles, batch, heads, C.c_longlong(n_bytes), group, int(fitted), out)
            return tuple(out)

        @staticmethod
        def score_cuts(batch, max_pages, min_pages, mean_bytes, rec_bytes):
            return bool(c.score_cuts(batch, max_pages, min_pages, mean_bytes, C.c_longlong(rec_bytes)))

        @staticmethod
        def score_cut(pages, most_pages, ulps=0, three_fit=False, reserve=0):
            chunks, sizes = (C.c_int * len(pages))(), (C.c_int * len(pages))()
            n = c.score_cut((C.c_int * len(pages))(*pages), len(pages), most_pages, int(three_fit), reserve, ulps, chunks, sizes)
            return n, list(chunks), list(sizes)

        @staticmethod
        def score_cut_grid(batch, max_pages, most_pages, three_fit=False, reserve=0):
            return c.score_cut_grid(batch, max_pages, most_pages, int(three_fit), reserve)

        @staticmethod
        def score_cut_reserve(batch, heads, mb, group, head_dim, bf16_means):
            return c.score_cut_reserve(batch, heads, C.c_longlong(mb << 20), group, head_dim, int(bf16_means))

        @staticmethod
        def extra_lds(splits, list_kb, own, page_size=16, head_dim=128, bf16=True):
            return c.extra_lds(int(bf16), head_dim, page_size, splits, C.c_longlong(list_kb << 10), own)

        @staticmethod
        def last_page_rule(cut, workgroups, last_pages, mb, group, fitted=False):
            return c.last_page_rule(cut, workgroups, last_pages, mb, group, int(fitted))

        even_tile, tile_stride, held_lds, dense_merge_alone = c.even_tile, c.tile_stride, c.held_lds, c.dense_merge_alone
        dense_chunks, dense_balances, lds = c.dense_chunks, c.dense_balances, c.lds
        uses_groups, score_cut_three_fit = c.uses_groups, c.score_cut_three_fit

        @staticmethod
        def whole(batch, heads, max_pages, top_k, mean_bytes=512, streams=0, page_bytes=8192):
            return bool(c.whole(batch, heads, max_pages, top_k, page_bytes, mean_bytes, streams))

        @staticmethod
        def dense_cut(pages, heads, max_pages):
            chunks = (C.c_int * len(pages))()
            return c.dense_cut((C.c_int * len(pages))(*pages), len(pages), heads, max_pages, chunks), list(chunks)
    return Lib


def test_every_plan_covers_its_list_and_stays_inside_the_workspace(lib):
    r = random.Random(1)
    for i in range(20000):
        batch, heads = r.choice([r.randint(1, 40), r.randint(1, 600)]), 1 << r.randint(0, 5)
        length = r.choice([r.randint(1, 64), r.randint(1, 2000), r.randint(1, 40000), r.randint(1 << 20, (1 << 31) - 1)])
        max_pages = r.choice([length, max(1, length // r.randint(1, 40)), length + r.randint(1, 9999) if length < 1 << 30 else length])
        page = r.choice([64, 128]) * r.choice([8, 16, 32]) * 2 * r.choice([2, 4])
        where = (batch, heads, length, max_pages, page)
        pps0, n0, rot0 = lib.most(batch * heads, length)
        slow = i % 2
        pps, n, rot = lib.plan(*where, slow)
        assert rot0 == 0 and 4 <= pps0 <= 256 and (n0 - 1) * pps0 < length <= n0 * pps0, where
        # every entry is visited, no chunk is empty by construction, and the partial results fit
        assert pps % 4 == 0 and (n - 1) * pps < length <= n * pps and n <= n0, where
        # a long row among short ones is never left to a few workgroups
        fits = n == 1 and min(length, max_pages) <= pps0 and length <= 4 * pps0
        assert pps <= pps0 + (MORE_BYTES // 4 if slow and n == 1 else MORE_BYTES) // page or fits, where
        assert rot == 0 or (1 <= rot <= batch and rot & (rot - 1) == 0 and 1 < n <= 65535), where
        assert (rot != 0) == (1 < n <= 65535 and (length > max_pages or batch * heads >= 256)), where


@pytest.mark.parametrize("batch,heads,length,max_pages,page,longest", [
    (32, 8, 1024, 1024, 8192, 256),    # ragged lists of 256 rows
    (32, 8, 8192, 8192, 8192, 256),    # padded lists of 256 rows
    (1, 8, 1024, 64, 8192, 16),        # a budget far above the pages of the sequence
    (4, 8, 1024, 125, 8192, 64),
    (2, 8, 741, 183, 32768, 24),
    (24, 8, 150, 150, 8192, 52),       # one long list among short ones
])
def test_lists_that_may_be_short_keep_chunks_of_the_finer_cut(lib, batch, heads, length, max_pages, page, longest):
    assert lib.plan(batch, heads, length, max_pages, page)[0] <= longest


@pytest.mark.parametrize("batch,heads,length,page,want", [
    (12, 8, 200, 8192, (40, 5)), (4, 4, 1024, 8192, (64, 16)), (1, 8, 1024, 8192, (32, 32)), (2, 8, 16, 8192, (16, 1)),
    (20, 8, 32, 8192, (32, 1)), (80, 8, 64, 4096, (64, 1)), (1, 8, 128, 8192, (4, 32))])
def test_full_lists_are_cut_into_equal_shares(lib, batch, heads, length, page, want):
    assert lib.plan(batch, heads, length, 1 << 20, page) == (*want, 0)


def test_dense_lists_are_cut_finely(lib):
    assert lib.most(128, 8192) == (256, 32, 0)   # at most 256 pages per chunk
    assert lib.most(8, 2048) == (32, 64, 0)      # 512 workgroups
    assert lib.most(300, 200) == (200, 1, 0)


def test_eight_heads_on_the_vector_units_are_cut_sooner(lib):
    assert lib.plan(2, 4, 16, 2048, 8192) == (16, 1, 0)
    assert lib.plan(2, 4, 16, 2048, 8192, 1) == (4, 4, 0)
    assert lib.plan(2, 4, 12, 2048, 8192, 1) == (12, 1, 0)


def test_score_tiles_are_powers_of_two_within_their_bounds(lib):
    r = random.Random(2)
    for _ in range(20000):
        batch, heads = r.choice([r.randint(1, 40), r.randint(1, 65535)]), 1 << r.randint(0, 5)
        most = r.choice([r.randint(1, 3000), r.randint(1, 70000), r.randint(1, 1 << 28)])
        least = r.choice([0, most, r.randint(0, most)])
        max_tile = 256 if heads <= 8 else 2048 // heads
        t = lib.tile(batch, heads, r.choice([64, 128]), most, least, max_tile)
        assert 8 <= t <= max_tile and t & (t - 1) == 0, (batch, heads, most, least)
        if t > 32:  # larger tiles only where the batch supplies full ones for every unit, or the grid is large anyway
            assert batch * (least // t) >= 256 or batch * -(-most // t) >= 4096, (batch, heads, most, least)


@pytest.mark.parametrize("batch,heads,head_dim,pages,want", [
    (4, 8, 128, 4096, 32), (16, 8, 128, 2048, 64), (4, 8, 128, 8192, 64), (8, 8, 64, 8192, 128), (30, 8, 128, 3000, 128),
    (16, 8, 128, 8192, 256), (1, 8, 128, 62501, 128), (3, 8, 128, 9000, 64), (1, 8, 64, 62501, 64), (4, 1, 128, 4096, 64),
    (8, 1, 128, 8192, 128), (1, 8, 128, 2048, 8)])
def test_score_tiles_of_even_batches(lib, batch, heads, head_dim, pages, want):
    assert lib.tile(batch, heads, head_dim, pages, pages) == want


def test_score_tiles_fitted_to_an_even_batch_stay_inside_their_bounds_and_leave_the_busiest_unit_less(lib):
    r = random.Random(6)
    fitted = 0
    for _ in range(20000):
        batch, heads = r.choice([1, r.randint(1, 40), r.randint(1, 65535)]), 1 << r.randint(0, 5)
        most = r.choice([r.randint(1, 3000), r.randint(1, 70000), r.randint(1, 1 << 28)])
        least = r.choice([0, most, r.randint(0, most), most - most // 10])
        max_tile = 256 if heads <= 8 else 2048 // heads
        old = lib.tile(batch, heads, 128, most, least, max_tile)
        t = lib.even_tile(old, batch, most, least, r.choice([128, 256, 512]), max_tile)
        assert 8 <= t <= max_tile and t % 8 == 0 and lib.tile_stride(t) in (t, 1 << t.bit_length())
        if t != old:
            fitted += 1
            assert least >= most - most // 8
            assert batch * -(-most // t) <= 768
            assert -(-batch * -(-most // t) // 256) * t < -(-batch * -(-most // old) // 256) * old
    assert fitted > 300


@pytest.mark.parametrize("batch,heads,pages,mean_bytes,want", [
    (1, 8, 9000, 512, 40), (5, 8, 2000, 512, 40), (60, 8, 300, 512, 80), (12, 8, 3125, 512, 152), (10, 8, 8192, 512, 168),
    (80, 8, 1000, 512, 168), (1, 8, 33000, 256, 72), (24, 8, 1700, 128, 56), (6, 16, 2500, 256, 32), (1, 8, 2048, 512, 8),
    (16, 8, 8192, 512, 256), (4, 8, 16384, 512, 128), (1, 8, 62501, 256, 128), (80, 8, 4096, 256, 256), (24, 8, 5000, 512, 240), (150, 8, 30, 512, 16),
    (30, 8, 3000, 256, 128)])
def test_score_tiles_fitted_to_even_batches(lib, batch, heads, pages, mean_bytes, want):
    most = 256 if heads <= 8 else 2048 // heads
    tile = lib.tile(batch, heads, 128 if mean_bytes > 128 else 64, pages, pages, most)
    assert lib.even_tile(tile, batch, pages, pages, mean_bytes, most) == want


@pytest.mark.parametrize("elem,head_dim,group,most", [(2, 64, 1, 7), (2, 64, 2, 6), (2, 64, 4, 5), (2, 64, 8, 4), (2, 128, 4, None), (4, 64, 8, None)])
def test_score_workgroups_per_unit_of_bf16_caches_of_64_channels(lib, elem, head_dim, group, most):
    lds = lib.held_lds(elem, head_dim, group)
    assert lds == 0 if most is None else most * lds <= 160 << 10 < (most + 1) * lds and 2048 <= lds


@pytest.mark.parametrize("cut,workgroups,last_pages,mb,group,want", [
    (0, 256, 2, 8, 4, 6), (0, 257, 2, 44, 8, 2), (0, 256, 32, 45, 4, 1), (0, 512, 32, 191, 4, 1), (0, 512, 32, 192, 4, 2),
    (0, 512, 257, 400, 4, 1), (0, 512, 24, 400, 8, 1), (1, 512, 64, 400, 4, 2), (1, 512, 64, 128, 8, 2), (1, 512, 64, 129, 8, 1)])
def test_who_renews_the_last_pages_of_a_step(lib, cut, workgroups, last_pages, mb, group, want):
    """1: the workgroup of its tile, 2: workgroups of their own, 6: those first in the grid."""
    assert lib.last_page_rule(cut, workgroups, last_pages, mb, group) == want


def test_cases_of_last_pages_take_the_routes_that_they_name(lib):
    """The steps on a GPU whose last pages are renewed in every way there is: where the rules that a launch asks send them."""
    from tests.test_gpu_parity import LAST_PAGE_CASES
    seen = set()
    for dtype, stats, heads, group, head_dim, page_size, pages, bound, top_k, renewed, from_groups in LAST_PAGE_CASES:
        bf16, mean_bytes, batch = dtype.itemsize == 2, head_dim * stats.itemsize, len(pages)
        least, page_bytes = min(pages) - 1, page_size * head_dim * 2 * dtype.itemsize  # full pages of the shortest sequence
        streams = batch * heads * min(top_k, bound) * page_bytes > 96 << 20
        fuses = lib.fuses_of(batch, heads, bound, top_k, page_size, head_dim, bf16)
        assert not (fuses and lib.whole(batch, heads, bound, top_k, mean_bytes, streams, page_bytes))
        assert ("step" if fuses else "own") == from_groups if lib.uses_groups(bound, top_k) else from_groups is None
        record, most = heads * mean_bytes + 128, 256 if heads <= 8 else 2048 // heads
        n_bytes = batch * bound * record
        if lib.score_cuts(batch, bound, least, mean_bytes, record):
            _, _, rule, _ = lib.score_grid(True, 512, batch, heads, n_bytes, group)
            route = "cut, tile" if rule == 1 else "cut"
        else:
            plain = lib.tile(batch, heads, head_dim, bound, least, most)
            tile = lib.even_tile(plain, batch, bound, least, mean_bytes, most)
            _, _, rule, _ = lib.score_grid(False, -(-bound // tile), batch, heads, n_bytes, group, tile != plain)
            route = {1: "tile", 2: "last", 6: "first"}[rule]
        assert route == renewed, (batch, heads, bound, route)
        seen.add((route, from_groups))
    assert {"first", "last", "tile", "cut", "cut, tile"} == {r for r, _ in seen} and {("cut", "step"), ("cut", "own"), ("last", "step"), ("last", "own")} <= seen


@pytest.mark.parametrize("mb,last_pages,group,want", [(45, 2, 4, 2), (100, 512, 1, 2), (100, 513, 4, 1), (191, 32, 8, 1), (400, 32, 4, 2), (44, 2, 4, 2)])
def test_last_pages_of_batches_with_a_fitted_tile_have_workgroups_of_their_own(lib, mb, last_pages, group, want):
    assert lib.last_page_rule(0, 468, last_pages, mb, group, True) == want
    assert lib.last_page_rule(0, 468, last_pages, mb, group) == (1 if 44 < mb < 192 else want)



@pytest.mark.parametrize("batch,heads,pages", [(40000, 1, 4), (65535, 1, 1), (32767, 1, 8), (32768, 1, 8), (21846, 8, 1), (13108, 16, 1),
                                               (7282, 32, 1), (65535, 32, 3), (65530, 4, 16384), (65535, 2, 120000), (1, 1, 1), (16, 8, 700)])
@pytest.mark.parametrize("group", [1, 8])
def test_score_grid_of_a_step_stays_within_the_extents_of_a_launch(lib, batch, heads, pages, group):
    """Up to 65535 sequences, of a page or more: the rows of the grid are no more than 65535, and there is a workgroup for every tile and,
    where last pages have their own, for every four heads of a last page."""
    most = 256 if heads <= 8 else 2048 // heads
    for least in (0, pages):
        for mean_bytes in (128, 256, 512):
            plain = lib.tile(batch, heads, 128 if mean_bytes > 128 else 64, pages, least, most)
            tile = lib.even_tile(plain, batch, pages, least, mean_bytes, most)
            x, y, rule, extra = lib.score_grid(False, -(-pages // tile), batch, heads, batch * pages * (heads * mean_bytes + 128), group, tile != plain)
            assert y <= 65535 and x == -(-pages // tile)
            if rule & 2:
                assert y == batch + extra and x * extra >= batch * -(-heads // 4)
            else:
                assert (y, rule, extra) == (batch, 1, 0)
    if batch <= 256:
        x, y, rule, extra = lib.score_grid(True, 512, batch, heads, 64 << 20, group)
        assert (x, y, rule, extra) == (512 + batch * -(-heads // 4), 1, 2, 512)


def test_score_chunks_of_a_batch_cut_by_its_lengths_cover_every_page_once_and_fit_the_launch(lib):
    """Batches of up to 256 sequences, empty ones among them, far below the launch's bound or at it, in one round or in many: a
    sequence has just the chunks that its pages fill, all alike and none empty, also if the reciprocals that the device divides with are two
    units in the last place off, and all have a workgroup, those left to last pages not counted."""
    r = random.Random(4)
    rounds = set()
    for _ in range(20000):
        batch, most = r.choice([3, 64, 65, 256, r.randint(3, 256)]), r.choice([64, 128, 256])
        three_fit, reserve = r.choice([(True, 0), (False, 0), (False, batch), (False, 2 * batch), (False, 8 * batch)])
        bound = r.choice([8, r.randint(1, 500), r.randint(1, 70000), 1 << 20])
        if not -(-bound // 8) * batch <= 1 << 22:
            continue
        top = r.choice([1, min(9, bound), bound, r.randint(1, bound)])
        pages = [r.choice([0, min(top, 1), top, r.randint(0, top), r.randint(0, top)]) for _ in range(batch)]
        chunk, chunks, sizes = lib.score_cut(pages, most, 0, three_fit, reserve)
        assert chunk % 8 == 0 and 8 <= chunk <= most, (batch, most, chunk)
        assert chunks == [-(-n // chunk) for n in pages], (batch, most, chunk)
        assert sum(chunks) <= lib.score_cut_grid(batch, bound, most, three_fit, reserve), (batch, bound, most)
        for n, parts, size in zip(pages, chunks, sizes):
            assert 8 * size <= chunk and (parts - 1) * 8 * size < n <= parts * 8 * size or n == parts == 0, (n, parts, size)
        rounds.add(-(-sum(chunks) // 512))
        for ulps in (-2, 2):
            assert lib.score_cut(pages, most, ulps, three_fit, reserve) == (chunk, chunks, sizes), (batch, most, chunk)
    assert {1, 2, 3, 40} <= rounds


@pytest.mark.parametrize("group,head_dim,bf16_means,elem,batch,want", [
    (8, 128, 1, 2, 3, 1), (8, 128, 1, 4, 63, 0), (8, 128, 1, 4, 64, 1), (8, 128, 0, 2, 64, 0), (4, 128, 1, 2, 64, 0), (8, 64, 1, 2, 64, 0)])
def test_batches_of_eight_heads_that_are_cut_for_three_workgroups_to_a_unit(lib, group, head_dim, bf16_means, elem, batch, want):
    assert lib.score_cut_three_fit(group, head_dim, bf16_means, elem, batch) == want


def test_score_chunks_and_last_pages_run_at_the_same_time_where_two_workgroups_fit_a_unit(lib):
    """Eight heads on fp32 means: the chunks of one round and the workgroups of the last pages are no more than 512."""
    assert lib.score_cut_reserve(24, 8, 101, 8, 128, False) == 48
    assert lib.score_cut_reserve(24, 8, 101, 8, 128, True) == lib.score_cut_reserve(24, 8, 101, 4, 128, False) == 0
    assert lib.score_cut_reserve(24, 8, 129, 8, 128, False) == 0  # in the tile
    r = random.Random(5)
    for _ in range(2000):
        batch = r.randint(3, 100)
        reserve = 2 * batch
        pages = [r.randint(0, 4000) for _ in range(batch)]
        _, chunks, _ = lib.score_cut(pages, 256, 0, False, reserve)
        need = -(-sum(-(-n // 8) for n in pages) // 32) + batch + reserve
        assert sum(chunks) + reserve <= 512 * -(-need // 512)


@pytest.mark.parametrize("batch,max_pages,min_pages,mean_bytes,rec_bytes,want", [
    (16, 4096, 300, 512, 4224, True), (2, 30000, 300, 512, 4224, False), (3, 30000, 300, 512, 4224, True), (256, 4096, 1, 512, 4224, True),
    (257, 4096, 1, 512, 4224, False), (15, 1500, 0, 512, 4224, False), (16, 1500, 0, 512, 4224, True), (16, 700, 0, 512, 4224, False),
    (16, 4096, 0, 128, 1152, False), (16, 6000, 0, 128, 1152, True), (3, (1 << 20) + 1, 0, 512, 4224, False),
    (40, 1 << 20, 0, 512, 4224, False), (16, 1500, 749, 512, 4224, True), (16, 1500, 750, 512, 4224, False),
    (16, 4096, 2048, 512, 4224, True), (16, 4096, 3584, 512, 4224, True), (16, 4096, 3585, 512, 4224, False), (7, 9000, 5000, 512, 4224, False),
    (8, 9000, 5000, 512, 4224, True), (16, 20000, 10000, 128, 1152, False), (16, 4096, 4096, 512, 4224, False),
    (16, 1000, 0, 512, 4224, False), (16, 1060, 0, 512, 4224, True), (16, 1000, 1, 512, 4224, True), (64, 380, 0, 256, 2176, False), (64, 395, 0, 256, 2176, True),
    (64, 195, 60, 512, 4224, True), (65, 195, 60, 512, 4224, True), (256, 127, 1, 512, 4224, False), (256, 128, 1, 512, 4224, True),
    (100, 237, 0, 512, 4224, False), (100, 240, 0, 512, 4224, True), (100, 237, 20, 512, 4224, True)])
def test_batches_whose_scores_are_cut_by_the_lengths(lib, batch, max_pages, min_pages, mean_bytes, rec_bytes, want):
    assert lib.score_cuts(batch, max_pages, min_pages, mean_bytes, rec_bytes) == want


@pytest.mark.parametrize("head_dim,page_size,key_bytes,bf16_means,least_mb", [
    (128, 16, 2, True, 144), (64, 32, 2, True, 144), (128, 16, 4, False, 144), (128, 16, 4, True, 144),
    (128, 8, 2, True, 288), (64, 16, 2, True, None), (64, 8, 2, True, None), (128, 16, 2, False, None),
    (128, 32, 2, False, None)])
def test_statistics_are_written_past_the_caches_where_that_measured_faster(lib, head_dim, page_size, key_bytes, bf16_means,
                                                                           least_mb):
    assert not lib.bulk(least_mb or 1 << 20, head_dim, page_size, key_bytes, bf16_means)
    assert lib.bulk((least_mb or 1 << 20) + 1, head_dim, page_size, key_bytes, bf16_means) == (least_mb is not None)


@pytest.mark.parametrize("batch,heads,pages,top_k,want", [
    (1, 8, 4096, 256, True), (1, 8, 4097, 256, False), (1, 8, 4097, 170, True), (1, 8, 6144, 256, True), (1, 8, 6143, 256, False),
    (1, 8, 32768, 256, True), (1, 8, 32769, 256, False), (16, 8, 8192, 256, True), (17, 8, 8192, 256, False), (1, 8, 4096, 257, False), (1, 8, 512, 200, True), (1, 8, 513, 200, False),
    (80, 8, 4096, 64, True), (24, 8, 1000, 64, True), (31, 8, 4096, 64, False)])
def test_steps_that_select_and_attend_in_one_kernel(lib, batch, heads, pages, top_k, want):
    assert lib.fuses(batch, heads, pages, top_k) == want


@pytest.mark.parametrize("batch,pages,top_k,page_size,head_dim,bf16,want", [
    (16, 4096, 128, 16, 128, True, True), (17, 4096, 128, 16, 128, True, True), (31, 4096, 64, 16, 128, True, True),
    (31, 2732, 128, 32, 128, True, True), (31, 4097, 64, 16, 128, True, False), (17, 4096, 257, 16, 128, True, False),
    (20, 4096, 128, 8, 128, True, False), (16, 4096, 128, 8, 128, True, True), (20, 2600, 128, 8, 128, True, True),
    (20, 4096, 128, 8, 64, True, True), (20, 4096, 128, 8, 128, False, True), (48, 1000, 60, 16, 128, True, True)])
def test_cut_rows_are_selected_from_in_every_workgroup_up_to_a_number_of_them(lib, batch, pages, top_k, page_size, head_dim, bf16, want):
    assert lib.fuses_of(batch, 8, pages, top_k, page_size, head_dim, bf16) == want


def test_uncut_rows_with_long_lists_have_two_workgroups_to_a_unit(lib):
    unit = 160 << 10
    for own in (18528, 37056, 40224, 48544, 57344, 70000):  # of the kernels, and more than any has
        for kb in (512, 768, 4096):
            total = own + lib.extra_lds(1, kb, own)
            assert 3 * total > unit and (2 * total <= unit or total == own)
    for other in (lib.extra_lds(2, 4096, 37056), lib.extra_lds(1, 511, 37056), lib.extra_lds(1, 4096, 37056, page_size=8),
                  lib.extra_lds(1, 4096, 20000, head_dim=64), lib.extra_lds(1, 4096, 20000, bf16=False)):
        assert other == 0


def test_chunks_of_many_dense_rows_are_merged_by_one_wave(lib):
    assert [lib.dense_merge_alone(n) for n in (2, 64, 127, 128, 256)] == [0, 0, 0, 1, 1]


def test_chunks_of_a_balanced_dense_batch_fit_the_workspace_and_leave_room_to_cut(lib):
    r = random.Random(3)
    seen = 0
    for _ in range(20000):
        batch, heads, pages = r.randint(1, 70), 1 << r.randint(0, 5), r.choice([r.randint(1, 500), r.randint(1, 70000)])
        if not lib.dense_balances(batch, heads, pages, r.choice([2048, 8192, 32768])):
            continue
        seen += 1
        rows, n = batch * heads, lib.dense_chunks(batch * heads, pages)
        assert 2 <= batch <= 64 and rows < n <= rows * lib.most(rows, pages)[1], (batch, heads, pages)
        assert n % 512 == 0 or n == rows * lib.most(rows, pages)[1], (batch, heads, pages)
    assert seen > 2000
    assert not lib.dense_balances(4, 8, 383, 8192) and lib.dense_balances(4, 8, 384, 8192)  # 96 MB
    assert not lib.dense_balances(1, 8, 100000, 8192) and not lib.dense_balances(33, 8, 4096, 8192)


@pytest.mark.parametrize("elem_bytes,head_dim,group,most", [(2, 128, 4, 3), (4, 64, 1, 7), (4, 64, 2, 6), (2, 128, 1, None), (2, 128, 8, None),
                                                            (2, 64, 4, None), (4, 128, 4, None), (4, 64, 4, None)])
def test_score_workgroups_per_unit_where_the_registers_allow_one_too_many(lib, elem_bytes, head_dim, group, most):
    """The LDS of a compute unit (160 KB, handed out in pieces of at most 2 KB) holds exactly `most` workgroups of a launch
    that could otherwise be on the chip at once; a workgroup never gets less than its scores take."""
    for scores in (32, 4096, 32768):
        for workgroups in [1, 4096] + ([] if most is None else [256 * most, 256 * most + 1, 256 * (most + 1)]):
            got = lib.lds(scores, elem_bytes, head_dim, group, workgroups)
            assert got >= scores
            if most is None or workgroups > 2560 or workgroups <= 256 * most:
                assert got == scores
            elif scores < 8192:
                assert -(-got // 2048) * 2048 * most <= 160 << 10 < got // 128 * 128 * (most + 1)


def test_the_cut_of_a_dense_batch_gives_every_chunk_a_slot(lib):
    """Rows of any mixture of lengths: no more chunks than workgroups that look for one and than slots of the workspace, at
    least one per row that has pages, none longer than the share that is certain to fit (a 64th more for the search and a
    rounding to whole pages), and no more of them than a chunk of four pages (one per wave) and one."""
    r = random.Random(5)
    seen = 0
    while seen < 4000:
        batch, heads = r.randint(2, 64), 1 << r.randint(0, 5)
        bound = r.choice([r.randint(2, 3000), r.randint(2, 70000)])
        if not lib.dense_balances(batch, heads, bound, r.choice([2048, 8192, 32768])):
            continue
        seen += 1
        kind = r.randint(0, 4)
        longest = r.choice([bound, max(1, bound // r.randint(1, 300))])
        pages = [r.randint(0, longest) if kind == 0 else longest if kind == 1 else max(1, int(longest ** r.random())) if kind == 2 else
                 longest - r.randint(0, min(3, longest)) if kind == 3 else r.randint(0, min(4, longest)) for _ in range(batch)]
        if kind == 4:
            pages[r.randrange(batch)] = longest
        looking, chunks = lib.dense_cut(pages, heads, bound)
        where = (pages, heads, bound, looking, chunks)
        rows, total = batch * heads, sum(pages) * heads
        assert sum(chunks) * heads <= looking <= lib.dense_chunks(rows, bound), where
        slots = min(max(total // (512 * 256), 1) * 512, lib.dense_chunks(rows, bound))
        even = len(set(pages)) == 1
        for p, n in zip(pages, chunks):
            assert (n >= 1) == (p > 0), where
            if p:
                length = -(-p // n)
                assert n <= p // 4 + 1, where
                share = p if even and n == slots // rows else total / (slots - rows)
                assert length <= max(4, share * 65 / 64 + 1 + 4 * even), where
    # a long sequence among many short ones gets nearly all slots
    _, chunks = lib.dense_cut([6250] + [4] * 30, 8, 6250)
    assert chunks[0] * 8 > 400 and chunks[1:] == [1] * 30


def test_steps_that_select_from_group_maxima_are_selections_that_have_them(lib):
    """A fused step of more pages than a row in registers is selected from the group maxima, which the score kernel only
    leaves where select_uses_groups says so; rows that are scored in the same kernel are short enough for its registers."""
    r = random.Random(7)
    fused = 0
    for _ in range(50000):
        batch, heads, pages = r.randint(1, 90), 1 << r.randint(0, 5), r.choice([r.randint(1, 5000), r.randint(1, 140000)])
        top_k = r.choice([r.randint(1, 300), max(1, pages // 24 + r.randint(-2, 2))])
        if lib.fuses(batch, heads, pages, top_k):
            fused += pages > 4096
            assert pages <= 4096 or (lib.uses_groups(pages, top_k) and pages <= 32768), (batch, heads, pages, top_k)
            assert top_k <= 256
        if lib.uses_groups(pages, top_k):
            assert 4096 < pages <= 131072 and 24 * top_k <= pages and top_k <= 1280
    assert fused > 500
    for mean_bytes, most in ((256, 384), (512, 256)):
        assert lib.whole(1, 8, most, 64, mean_bytes) and not lib.whole(1, 8, most + 1, 64, mean_bytes)
        assert not lib.whole(1, 8, 8, 8, mean_bytes, streams=1)


@pytest.mark.parametrize("batch,top_k,want", [(16, 64, True), (17, 64, False), (24, 64, False), (24, 16, True), (16, 200, True), (17, 200, True),
                                              (20, 200, False), (80, 8, True)])
def test_steps_scored_in_every_workgroup_fit_the_chip_at_once_or_are_not_cut(lib, batch, top_k, want):
    assert lib.whole(batch, 8, 250, top_k) == want
