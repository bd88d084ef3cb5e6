"""The rules that cut a launch into workgroups, over the sizes they are asked for."""
from tests.host_rules import in_ring, tiles_per_wave


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
