"""The rules that cut a launch into workgroups, over the sizes they are asked for."""
from tests.host_rules import tiles_per_wave


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
