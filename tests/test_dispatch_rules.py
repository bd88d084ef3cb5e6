"""The rules that cut a launch into workgroups, over the sizes they are asked for."""
from tests.host_rules import in_ring, key_ranges, tile_of_walk, tiles_per_wave


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
