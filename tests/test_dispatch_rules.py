"""The rules that cut a launch into workgroups, over the sizes they are asked for."""
from tests.host_rules import (f32_one_launch, f32_waves, in_ring, key_ranges, stage1_one_launch, tile_of_walk, tiles_per_wave,
                              walk_start, walk_ticks)


def _cost(T, n_tiles, tpw):
    """Rounds of 512 workgroups at 4 (a last one with at most 256: 3), each as long as its tiles and six more."""
    wgs = T * -(-n_tiles // (4 * tpw))
    rest = wgs % 512
    return (4 * (wgs // 512) + (4 if rest > 256 else 3 if rest else 0)) * (tpw + 6)


def test_tiles_per_wave():
    for T in (1, 2, 3, 31, 32, 64, 77, 130, 200, 255, 256, 1000, 2000, 65536, 1 << 20):
        for n in (1, 4, 5, 8, 16, 64, 65, 129, 256, 511, 512, 2000, 2048):
            tpw = tiles_per_wave(T, n)
            costs = [_cost(T, n, t) for t in range(1, 17)]
            assert 1 <= tpw <= 16 and costs[tpw - 1] == min(costs), (T, n, tpw)
            if T >= 65536:         # many queries: no more workgroups than tiles of 64 need, so the grid stays legal
                assert -(-n // (4 * tpw)) == -(-n // 64), (T, n, tpw)


def test_tiles_per_wave_at_the_sizes_its_figures_are_for():
    sizes = {(1, 256): 1, (32, 256): 4, (130, 256): 10, (200, 128): 16, (200, 256): 13, (255, 512): 16}
    assert {s: tiles_per_wave(*s) for s in sizes} == sizes


def test_bins_in_the_tile_rings():
    # two or three workgroups per CU: where a third saves a round (one of 512 queries turns into one of 768)
    for T, want in ((1, False), (512, False), (513, True), (768, True), (769, False), (1024, False), (1025, True),
                    (65536, True)):
        assert in_ring(T, 16384, False, True, 2, 3) == want, T
    # three or four
    for T, want in ((768, False), (769, True), (1024, True), (1025, False), (1537, True), (2100, False), (65536, True)):
        assert in_ring(T, 16384, False, True, 3, 4) == want, T
    assert not in_ring(65536, 16384, False, True, 3, 3)          # no workgroup more
    # bf16 keys of one long sequence; fp8 keys and packed streams at any length
    assert in_ring(16384, 49152, False, False, 2, 3) and not in_ring(16384, 49184, False, False, 2, 3)
    assert in_ring(16384, 1 << 20, True, False, 2, 3) and in_ring(16384, 1 << 20, False, True, 2, 3)


def test_key_ranges_of_the_prefill_scoring_kernel():
    for T in (1, 64, 77, 100, 256, 777, 1024, 2048, 4096, 8184):
        for last in (0, 1, 127, 128, 129, 5000, 65536, 1 << 20):
            for first in (0, last // 2, max(0, last - T), last):
                s = key_ranges(T, first, last)
                assert 1 <= s <= 32 and (s == 1 or s <= -(-last // 128)), (T, first, last, s)     # no empty range
    assert key_ranges(8192, 0, 65536) == 1                       # four rounds by themselves
    # queries at the end of a long context fill the CUs as often as they can be cut evenly
    assert [key_ranges(T, 64512, 65536) for T in (1024, 512, 256)] == [2, 4, 8]
    assert key_ranges(3000, 1, 3000) == 1                        # a triangle: the short queries fill the second round
    # what is seen counts, not the array's length: 300 pooled keys, whatever the cache was made for
    assert key_ranges(1500, 253, 300) == 1


def test_walks_cover_a_waves_tiles_and_stay_in_the_block_list():
    # the fused Stage 2: every lane of every wave looks a tile up in the query's m block ids, also lanes and waves without one
    for n_waves, m, per_block in ((4, 2, 1), (4, 3, 1), (4, 2, 2), (4, 5, 1), (4, 7, 4), (8, 2, 1), (8, 3, 2), (8, 257, 1), (4, 64, 4)):
        for used in sorted({0, 1, m - 1, m}):
            tiles = used * per_block
            for wave in range(n_waves):
                nj = max(0, -(-(tiles - wave) // n_waves))
                for j0 in sorted({0, nj // 2 // 2 * 2, max(0, nj - 2)} if nj % 2 == 0 else {0}):
                    at = [tile_of_walk(j, nj, j0, wave, n_waves) for j in range(max(64, nj))]
                    assert all(0 <= v < m * per_block for v in at), (n_waves, m, per_block, used, wave, at)
                    assert sorted(at[:nj]) == list(range(wave, tiles, n_waves)), (n_waves, m, used, wave)


def test_fp32_rows_in_one_launch_only_where_it_is_the_faster():
    # (queries, candidates, heads, d), us in two launches, us in one
    measured = [
        ((1024, 256, 4, 64), 17.3, 13.4), ((1024, 512, 4, 64), 25.9, 18.6), ((700, 512, 4, 64), 21.4, 18.3), ((256, 32, 4, 64), 10.9, 9.9),
        ((4096, 48, 8, 4), 16.3, 11.4), ((4096, 65, 2, 16), 18.0, 12.9), ((16000, 64, 3, 20), 41.3, 29.4), ((256, 257, 64, 32), 37.2, 26.0),
        ((700, 256, 3, 64), 28.0, 14.0), ((16000, 64, 6, 64), 108.7, 60.0), ((2048, 65, 3, 96), 32.6, 16.4), ((6000, 256, 3, 96), 356.2, 63.0),
        ((1024, 512, 16, 96), 99.4, 60.6), ((4096, 48, 8, 128), 36.6, 24.8), ((512, 320, 8, 128), 29.9, 20.7),
        ((2048, 512, 16, 128), 237.3, 134.5), ((4096, 400, 12, 128), 285.3, 191.9), ((300, 400, 8, 256), 56.8, 35.9), ((3000, 512, 4, 512), 353.9, 201.6),
        ((400, 320, 9, 512), 125.5, 72.7), ((2048, 512, 3, 512), 1488.0, 182.4), ((100, 512, 128, 32), 66.0, 45.4),
        ((2048, 48, 128, 4), 22.0, 37.8), ((3000, 512, 4, 4), 17.4, 27.8), ((768, 512, 32, 8), 17.9, 31.3), ((16000, 192, 5, 12), 51.2, 83.5),
        ((16000, 512, 24, 12), 147.7, 374.1), ((2048, 192, 8, 16), 14.6, 20.8), ((6000, 512, 8, 16), 39.2, 78.1), ((1, 64, 64, 16), 13.3, 28.5),
        ((100, 20, 128, 16), 25.0, 52.8), ((6000, 32, 128, 16), 63.7, 485.0), ((512, 129, 32, 20), 14.4, 21.3), ((400, 64, 24, 24), 12.8, 18.4),
        ((600, 128, 24, 28), 15.7, 21.9), ((300, 129, 128, 36), 37.9, 66.6), ((4096, 65, 32, 48), 53.2, 101.2), ((3000, 128, 128, 48), 174.5, 522.7),
        ((600, 20, 128, 64), 52.3, 82.9), ((100, 192, 128, 96), 80.5, 120.1), ((1024, 64, 64, 128), 77.2, 121.7), ((700, 64, 24, 256), 44.7, 61.0),
        ((2048, 32, 9, 512), 67.2, 100.6), ((700, 96, 24, 512), 125.7, 185.2)]
    for call, two, one in measured:
        assert f32_one_launch(*call) == (one < two), call
    assert not f32_one_launch(1, 64, 128, 4) and f32_one_launch(1 << 22, 512, 4, 64)     # the ends of what a call may hold
    for T in (1, 63, 768, 769, 2048, 2049, 1 << 22):
        for n in (1, 63, 64, 65, 128, 129, 256, 257, 512):
            waves = f32_waves(T, n)
            assert waves in (1, 2, 4, 8) and (waves == 1 or 64 * waves // 2 < n), (T, n, waves)   # no wave without a candidate of its own


def test_walks_begin_in_step():
    # the waves of a workgroup begin at the same one of their tiles, at an even one, and never in a walk that is odd
    for n_waves in (4, 8):
        for n_tiles in list(range(1, 140)) + [244, 256, 500, 512]:
            njs = {max(0, -(-(n_tiles - w) // n_waves)) for w in range(n_waves)}
            seen = {walk_start(n_tiles, n_waves, now, 200) for now in [0, 199, 200, 12345, 0xffffffff] + [200 * i for i in range(70)]}
            if len(njs) > 1 or min(njs) % 2:
                assert seen == {0}, (n_tiles, n_waves)
            else:
                assert seen == set(range(0, min(njs), 2)), (n_tiles, n_waves)


def test_walks_only_over_more_keys_than_an_l2_holds():
    assert walk_ticks(4 << 20, 0) == 0 and walk_ticks(4 << 20, 1) == 0
    assert walk_ticks((4 << 20) + 1, 0) == 200 and walk_ticks((1 << 31) - 1, 1) == 160


def test_stage1_in_one_launch():
    # up to a query per CU: whatever the select holds; beyond: two rounds of 512 (64 heads) or 768 (32), rows of a one-wave select
    for H, two_rounds in ((64, 1024), (32, 1536)):
        assert stage1_one_launch(1, 1, H) and stage1_one_launch(256, 8192, H) and not stage1_one_launch(256, 8193, H)
        assert stage1_one_launch(257, 512, H) and not stage1_one_launch(257, 513, H)
        assert stage1_one_launch(two_rounds, 512, H) and not stage1_one_launch(two_rounds + 1, 512, H)
        assert not stage1_one_launch(1 << 22, 1, H)
