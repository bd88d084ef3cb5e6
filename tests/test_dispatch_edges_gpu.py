"""Parity at the edges of the size-dependent dispatch rules: each case sits where one kernel hands over
to another, or where the way a kernel divides its work changes."""
import numpy as np
import pytest

from paper_2603_28458_amd import workloads as W
from tests.host_rules import in_ring, key_ranges, tiles_per_wave
from tests.parity import run_and_check, sample_queries

pytestmark = pytest.mark.gpu


def _run(wl, n=24, **kw):
    print(f"\n[parity] {wl.name}: T={wl.T} H={wl.H} B={wl.B} m={wl.m} k={wl.k} k={wl.k_dtype} n_seq={wl.n_seq} "
          f"s_max={wl.s_max} seed={wl.seed}", flush=True)
    return run_and_check(wl, queries=sample_queries(wl, n), **kw)


@pytest.mark.parametrize("T,L,s_max,k_dtype,ranges", [
    (64, 9001, None, "bf16", 32), (71, 4097, None, "fp8_e4m3", 28), (257, 30000, None, "bf16", 7), (1000, 6400, None, "fp8_e4m3", 2),
    (2055, 2055, None, "bf16", 2), (3000, 4000, None, "bf16", 1), (300, 700, 20000, "fp8_e4m3", 6)])
def test_key_ranges_of_the_prefill_scoring_kernel(T, L, s_max, k_dtype, ranges):
    # the dense scoring kernel (flat indexer, Stage 1 of a chunk) cuts the keys of 8 queries into ranges of
    # 128-key tiles: by how many groups of 8 there are and what their queries see, whatever the cache was made
    # for; uneven ranges, ranges past a short prefix
    assert key_ranges(T, L - T + 1, L) == ranges
    wl = W.make_workload(f"ranges{T}", seq_len=L, T=T, H=64, d=128, B=32, m=20, k=min(512, L), q_dtype="bf16",
                         k_dtype=k_dtype, s_max=s_max, seed=400 + T)
    _run(wl)


@pytest.mark.parametrize("k_dtype,H,d", [("bf16", 64, 128), ("fp8_e4m3", 32, 128), ("f32", 4, 64)])
@pytest.mark.parametrize("packed", [False, True])
def test_queries_that_keep_everything(k_dtype, H, d, packed):
    # visible blocks around the block budget and visible tokens around the token budget, with sequences of
    # their own (two-kernel Stage 2 below 256 queries, fused above) and in a packed stream whose starts are
    # no multiples of the block; a sequence of one token, one of exactly k, one of exactly m * B
    B, m, k = 32, 8, 130
    qd = "f32" if k_dtype == "f32" else "bf16"
    for lens in ([1, 130, 70], [256, 1, 131, 130, 400, 33]):
        wl = W.make_workload(f"all_{k_dtype}_{packed}_{len(lens)}", n_seq=len(lens), seq_len=lens, T=sum(lens), H=H, d=d,
                             B=B, m=m, k=k, q_dtype=qd, k_dtype=k_dtype, mode="varlen", seed=420)
        _run(W.pack(wl) if packed else wl, n=10000)


def _workspaces(op, Q, K, B, m, k):
    """Workspaces a call may be handed: full of large scores, of NaN, of the mark that an earlier call leaves
    in a row it did not score."""
    import torch
    from paper_2603_28458_amd import hisa

    n = max(256, hisa.hisa_workspace_bytes(op, Q, K, B, m, k))
    for word in (0x7f7fffff, -1, 0x7f800001):
        yield torch.full((n // 4,), word, dtype=torch.int32, device="cuda").view(torch.uint8)


def _routes_agree(Q, K, blocks, B, m, k):
    """The ids must not depend on whether the scores are asked for (which scores and selects every row), nor
    on what the workspace holds."""
    from paper_2603_28458_amd import hisa

    general = hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k, want_topk_scores=True)[0].cpu().numpy()
    for ws in _workspaces(hisa.OP_TOKEN_REFINE_TOPK, Q, K, B, m, k):
        short = hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k, ws=ws)[0].cpu().numpy()
        assert np.array_equal(short, general), np.nonzero((short != general).any(1))[0]


@pytest.mark.parametrize("T", [200, 300])        # two-kernel and fused Stage 2 (fp32: two-kernel)
@pytest.mark.parametrize("k_dtype,H,d", [("bf16", 64, 128), ("fp8_e4m3", 32, 128), ("f32", 4, 64)])
def test_rows_kept_whole_equal_the_scored_rows(k_dtype, H, d, T):
    # visible tokens and blocks below the budgets, but block lists that Stage 1 does not write (any order,
    # gaps, repeats, blocks out of sight or out of range), and scores of -inf, which drop a block in Stage 1
    # and a token in the two-kernel Stage 2
    import torch
    from paper_2603_28458_amd import hisa

    B, m, k = 32, 12, 320
    f32 = k_dtype == "f32"
    wl = W.make_workload(f"whole_{k_dtype}_{T}", seq_len=T, T=T, H=H, d=d, B=B, m=m, k=k,
                         q_dtype="f32" if f32 else "bf16", k_dtype=k_dtype, seed=430)
    print(f"\n[routes] {wl.name}", flush=True)
    Q, K = hisa.to_device(wl)
    pd = hisa.HISA_F32 if f32 else hisa.HISA_BF16
    rng = np.random.default_rng(431)
    nb = -(-T // B)
    lists = np.full((T, m), -1, dtype=np.int32)
    for t in range(T):
        n = int(rng.integers(1, m + 1))
        kind = t % 4
        if kind == 0:
            lists[t, :n] = rng.integers(-1, nb, n)                  # repeats, gaps, any order
        elif kind == 1:
            lists[t, :n] = rng.permutation(m)[:n]                   # blocks past the query and past the array
        elif kind == 2:
            p = rng.permutation(t // B + 1)[:n]
            lists[t, :p.size] = np.sort(p)                          # ascending, not all of them
        else:
            p = np.arange(min(m, t // B + 3))
            lists[t, :p.size] = p                                   # ascending, past the query's own block
    _routes_agree(Q, K, torch.from_numpy(lists).cuda(), B, m, k)

    Q.w[::3, 1] = -np.inf
    Q.w[1::5, 0] *= -1.0
    pooled = hisa.hisa_pool_blocks(K, B, pooled_dtype=pd)
    short = hisa.hisa_block_score_topk(Q, K, pooled, pd, B, m)[0]
    general = hisa.hisa_block_score_topk(Q, K, pooled, pd, B, m, want_scores=True)[0]
    assert torch.equal(short, general)
    _routes_agree(Q, K, short, B, m, k)
    if k_dtype == "fp8_e4m3":
        Q.w.abs_()
        Q.w.clamp_(max=2.0)
        K.k_scale[:, ::7] = -np.inf
        _routes_agree(Q, K, short, B, m, k)
    # memory filled with ones: the pattern that marks a masked slot in the fused kernel
    Q.w.abs_()
    ones = torch.full((1,), -1, dtype=torch.int32, device="cuda").view(torch.float32)
    Q.w[::4, 2] = ones
    _routes_agree(Q, K, short, B, m, k)
    if k_dtype == "fp8_e4m3":
        Q.w[:] = 1.0
        K.k_scale[:, 5::9] = ones
        _routes_agree(Q, K, short, B, m, k)


@pytest.mark.parametrize("T,positions,packed", [(100, False, False), (600, False, False), (600, True, False), (600, False, True),
                                                (2100, False, False), (2100, False, True)])
@pytest.mark.parametrize("H", [64, 32])
def test_gates_that_refuse_the_direct_write_of_blocks(T, H, positions, packed):
    # every query sees at most m blocks, so nothing is scored unless a gate could make a score -inf or NaN; on each
    # route of Stage 1 (k_stage1_query, k_score_prefill, k_score_ranges by given positions and packed,
    # k_score_resident plain and packed) and in the single-launch call the blocks must be those of the scored
    # rows, whatever the workspace holds
    import torch
    from paper_2603_28458_amd import hisa

    B, m = 32, 80
    cut = [0, T // 3 + 5, T]
    lens = [b - a for a, b in zip(cut, cut[1:])] if packed else T
    wl = W.make_workload(f"gates{T}_{positions}_{packed}", n_seq=2 if packed else 1, seq_len=lens, T=T, H=H, d=128, B=B, m=m, k=64,
                         q_dtype="bf16", k_dtype="bf16", mode="varlen" if packed else "prefill", seed=470)
    Q, K = hisa.to_device(W.pack(wl) if packed else wl)
    if positions:
        Q.q_pos = torch.arange(T, dtype=torch.int32, device="cuda")
    print(f"\n[gates] T={T} H={H} positions={positions} packed={packed}", flush=True)
    pooled = hisa.hisa_pool_blocks(K, B)
    ones = torch.full((1,), -1, dtype=torch.int32, device="cuda").view(torch.float32)
    Q.w[::3, 1] = -np.inf
    Q.w[1::5, 0] *= -1.0
    Q.w[2::7, 3] = ones
    general = hisa.hisa_block_score_topk(Q, K, pooled, hisa.HISA_BF16, B, m, want_scores=True)[0].cpu().numpy()
    for ws in _workspaces(hisa.OP_BLOCK_SCORE_TOPK, Q, K, B, m, 0):
        short = hisa.hisa_block_score_topk(Q, K, pooled, hisa.HISA_BF16, B, m, ws=ws)[0].cpu().numpy()
        assert np.array_equal(short, general), np.nonzero((short != general).any(1))[0]
    one = hisa.hisa_indexer_topk(Q, K, pooled, hisa.HISA_BF16, B, m, 64, want_block_idx=True)[0].cpu().numpy()
    assert np.array_equal(one, general), np.nonzero((one != general).any(1))[0]


@pytest.mark.parametrize("T,M", [(1, 1), (256, 2), (256, 33), (1024, 130), (1025, 130), (300, 512), (256, 1019)])
@pytest.mark.parametrize("H", [64, 32])
def test_stage1_of_arrays_of_at_most_m_blocks(T, M, H):
    # positions in any order, none, past the sequence's end, and queries that see a part of it; gates that leave a query
    # unscored, or not, in which case blocks of infinite score drop out: m as large as the array, and a little larger
    import torch
    from paper_2603_28458_amd import hisa

    B, n = 32, 3
    print(f"\n[short arrays] T={T} M={M} H={H}", flush=True)
    g = torch.Generator().manual_seed(T + M)
    rng = np.random.default_rng(T + M)
    q, w = torch.randn((T, H, 128), generator=g), torch.rand((T, H), generator=g)
    q[:, 0, 1] = 3e38
    w[::2, 0] *= -1.0                                             # -inf where the pooled key's element 1 is large
    w[1::6, 5], w[3::6, 1] = float("nan"), 0.0
    pooled = torch.randn((n, M, 128), generator=g)
    pooled[:, :, 1] = 0.0
    pooled[:, M // 3:: 4, 1] = 3e38
    lens = np.array([M * B, max(1, M * B // 2 + 3), 1])
    seq = rng.integers(0, n, T)
    pos = rng.integers(-1, M * B + 40, T)
    lo = np.where(np.arange(T) % 4 == 0, rng.integers(0, np.maximum(1, np.minimum(pos, lens[seq] - 1) + 1)), 0)
    ints = lambda x: torch.from_numpy(x.astype(np.int32)).cuda()
    Q = hisa.Queries(q=q.bfloat16().cuda(), w=w.cuda(), dtype=hisa.HISA_BF16, q_seq=ints(seq), q_pos=ints(pos), q_lo=ints(lo))
    K = hisa.Keys(k=None, seq_len=ints(lens), dtype=hisa.HISA_BF16, n_seq=n, s_max=M * B, d=128)
    P = pooled.bfloat16().cuda()
    for m in (max(2, M), M + 5):
        got = hisa.hisa_block_score_topk(Q, K, P, hisa.HISA_BF16, B, m)[0].cpu().numpy()
        want = hisa.hisa_block_score_topk(Q, K, P, hisa.HISA_BF16, B, m, want_scores=True)[0].cpu().numpy()
        assert np.array_equal(got, want), np.nonzero((got != want).any(1))[0]
        unscored = (w >= 0).all(1).numpy()
        for t in range(T):
            last = min(pos[t], lens[seq[t]] - 1)
            ids = np.arange(lo[t] // B, last // B + 1) if last >= 0 else np.arange(0)
            kept = got[t][got[t] >= 0]
            assert np.isin(kept, ids).all() and (not unscored[t] or np.array_equal(kept, ids)), t


@pytest.mark.parametrize("H", [64, 32])
@pytest.mark.parametrize("T,q_pos0", [(2100, -1700), (4100, -3600)])
def test_flat_indexer_on_a_short_packed_stream(T, q_pos0, H):
    # at most 512 bf16 keys and 2048 queries or more at consecutive positions, with first visible positions: the
    # resident kernel (64, 32 or 8 queries per workgroup), against the same queries with their positions given
    # one by one, which go through the per-query kernel.  Queries before the stream, inside it, past its end
    import torch
    from paper_2603_28458_amd import hisa

    S, k = 480, 70
    wl = W.make_workload(f"flat_packed{T}", seq_len=S, T=S, H=H, d=128, B=32, m=4, k=k, q_dtype="bf16", k_dtype="bf16", seed=480)
    _, K = hisa.to_device(wl)
    g = torch.Generator().manual_seed(481)
    pos = q_pos0 + torch.arange(T)
    starts = torch.tensor([0, 7, 150, 151, 333, 1 << 20])
    lo = starts[torch.searchsorted(starts, pos.clamp(min=0), right=True) - 1].int().cuda()
    Q = hisa.Queries(q=torch.randn((T, H, 128), generator=g).bfloat16().cuda(), w=torch.rand((T, H), generator=g).cuda(),
                     dtype=hisa.HISA_BF16, q_pos0=q_pos0, q_lo=lo)
    print(f"\n[flat packed] T={T} H={H}", flush=True)
    ids, sc = hisa.dsa_flat_indexer_topk(Q, K, k, want_topk_scores=True)[:2]
    Q.q_pos = pos.int().cuda()
    want_ids, want_sc = hisa.dsa_flat_indexer_topk(Q, K, k, want_topk_scores=True)[:2]
    assert torch.equal(ids, want_ids) and torch.equal(sc, want_sc)
    ids = ids.cpu().numpy()
    assert (ids[: -q_pos0] == -1).all() and (ids[-q_pos0 : S - q_pos0, 0] >= 0).all()
    for t in range(-q_pos0, min(T, S - q_pos0), 11):
        row = ids[t][ids[t] >= 0]
        assert row.size == min(k, t + q_pos0 - int(lo[t]) + 1) and row[0] >= int(lo[t]) and row[-1] <= t + q_pos0


@pytest.mark.parametrize("T", [200, 300])
@pytest.mark.parametrize("k_dtype,H,d", [("bf16", 64, 128), ("fp8_e4m3", 32, 128), ("f32", 4, 64)])
def test_queries_before_position_zero_see_nothing(k_dtype, H, d, T):
    # as far before it as several blocks, where the first visible block must not come out below 0: every id is
    # -1, whatever is asked for; the queries after them are as they are without them
    from paper_2603_28458_amd import hisa

    B, m, k = 32, 8, 130
    f32 = k_dtype == "f32"
    wl = W.make_workload(f"before_{k_dtype}_{T}", seq_len=T, T=T, H=H, d=d, B=B, m=m, k=k, q_dtype="f32" if f32 else "bf16",
                         k_dtype=k_dtype, seed=435)
    Q, K = hisa.to_device(wl)
    pd = hisa.HISA_F32 if f32 else hisa.HISA_BF16
    pooled = hisa.hisa_pool_blocks(K, B, pooled_dtype=pd)
    Q.q_pos0 = -150
    for scores in (False, True):
        blocks = hisa.hisa_block_score_topk(Q, K, pooled, pd, B, m, want_scores=scores)[0]
        ids = hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k, want_topk_scores=scores)[0]
        got = [blocks, ids]
        if not f32:
            got += list(hisa.hisa_indexer_topk(Q, K, pooled, pd, B, m, k, want_block_idx=True, want_topk_scores=scores))[:2]
        for x in got:
            x = x.cpu().numpy()
            assert (x[:150] == -1).all() and (x[150:, 0] >= 0).all(), (scores, np.nonzero((x[:150] != -1).any(1))[0])


@pytest.mark.parametrize("k_dtype,T,m,k,wgs", [("bf16", 600, 128, 1024, 2), ("fp8_e4m3", 800, 128, 1024, 3),
                                               ("fp8_e4m3", 600, 256, 2048, 2)])
@pytest.mark.parametrize("kind", ["tied", "groups", "zero", "random"])
def test_top_k_bins_in_the_tile_rings(k_dtype, T, m, k, wgs, kind):
    # fused Stage 2 with 32 heads: the one-pass top-k's bins share the rings with the general select, which takes
    # over for a row it declines.  tied: 30 % of the scores are equal and the k-th is one of them: declined with
    # the bins full, for a crowded bin.  groups: about 20 equal scores around every rank, the k-th among them:
    # declined after the last check.  zero: every score equal: declined before a bin is touched
    import torch
    from paper_2603_28458_amd import hisa
    from tests.test_fine_select import expected_row, one_head_queries

    B, L = 32, 9000
    assert in_ring(T, L, False, k_dtype != "bf16", wgs, wgs + 1)      # (the form under test; T = 300 takes the other)
    wl = W.make_workload(f"rings_{k_dtype}_{m}", seq_len=L, T=T, H=32, d=128, B=B, m=m, k=k, q_dtype="bf16", k_dtype=k_dtype,
                         seed=440)
    if kind == "random":
        _run(wl, n=40)
        return
    rng = np.random.default_rng(441)
    if kind == "tied":
        level = np.where(rng.random(L) < 0.3, 128, np.where(rng.random(L) < 0.2, rng.integers(129, 256, L), rng.integers(0, 128, L)))
    else:
        level = rng.integers(0, 200 * m // 128, L) if kind == "groups" else np.zeros(L, np.int64)
    Q = hisa.Queries(**one_head_queries(32, T, {0: 1.0, 1: 256.0}), q_pos0=L - T)
    keys = torch.zeros((1, L, 128))
    scale = None
    if k_dtype == "bf16":
        keys[0, :, 0], keys[0, :, 1] = torch.from_numpy(level % 256).float(), torch.from_numpy(level // 256).float()
        keys = keys.bfloat16().cuda()
    else:
        keys[0, :, 0] = 1.0
        keys = keys.to(torch.float8_e4m3fn).view(torch.uint8).cuda()
        scale = torch.from_numpy(level).float()[None].cuda()
    K = hisa.Keys(k=torch.nn.functional.pad(keys, (0, 0, 0, -L % B)), seq_len=torch.tensor([L], dtype=torch.int32).cuda(),
                  dtype=hisa.DTYPE_CODE[k_dtype], k_scale=None if scale is None else torch.nn.functional.pad(scale, (0, -L % B)))
    print(f"\n[rings] {k_dtype} m={m} {kind}", flush=True)
    lists = np.sort(np.argsort(rng.random((T, (L - T) // B)), 1)[:, :m], 1).astype(np.int32)
    blocks = torch.from_numpy(lists).cuda()
    got = hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k)[0]
    # the two-kernel path, which keeps its bins apart
    want = hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k, want_cand_scores=True)[0]
    assert torch.equal(got, want)
    got = got.cpu().numpy()
    for t in range(0, T, 7):
        tok = (lists[t][:, None] * B + np.arange(B)).ravel()
        assert np.array_equal(got[t], expected_row(level[tok], tok, k)), t


@pytest.mark.parametrize("n_seq,B,m,k_dtype,H,tpw", [
    (1, 32, 20, "bf16", 64, 1), (65, 32, 33, "fp8_e4m3", 64, 3), (3, 32, 250, "fp8_e4m3", 32, 1), (64, 64, 32, "bf16", 64, 4),
    (130, 32, 66, "bf16", 32, 6), (32, 128, 125, "bf16", 64, 8), (130, 128, 64, "fp8_e4m3", 64, 10),
    (130, 32, 128, "bf16", 64, 11), (255, 32, 191, "fp8_e4m3", 32, 12), (200, 128, 64, "bf16", 32, 13),
    (200, 32, 128, "fp8_e4m3", 64, 16), (255, 64, 128, "bf16", 64, 16)])
def test_tiles_per_wave_of_a_decode_batch(n_seq, B, m, k_dtype, H, tpw):
    # Stage 2 below 256 queries: the number of tiles a wave walks follows from the queries and the candidates;
    # lengths of which some leave fewer blocks than m, so that the last workgroups of a query have idle waves
    assert tiles_per_wave(n_seq, m * B // 32) == tpw
    L = m * B + 300
    wl = W.make_workload(f"tpw{n_seq}", n_seq=n_seq, seq_len=[L - (37 * i) % (L // 2) for i in range(n_seq)], T=n_seq, H=H,
                         d=128, B=B, m=m, k=min(300, B * m), q_dtype="bf16", k_dtype=k_dtype, mode="decode", seed=450)
    _run(wl, n=8)


@pytest.mark.parametrize("T,H", [(2051, 64), (3073, 32), (6145, 64), (12290, 32)])
@pytest.mark.parametrize("packed", [False, True])
def test_queries_per_wave_of_the_resident_scoring_kernel(T, H, packed):
    # Stage 1 up to 512 blocks: 1, 2, 4 and 8 queries per wave, the last workgroup with one query or a few; in a
    # packed stream workgroups with queries of two sequences, whose blocks start in the middle of a sub-tile
    cut = [0, 700, 701, T // 2 + 13, T]
    lens = [b - a for a, b in zip(cut, cut[1:])] if packed else T
    wl = W.make_workload(f"resident{T}_{packed}", n_seq=4 if packed else 1, seq_len=lens, T=T, H=H, d=128, B=32, m=9,
                         k=256, q_dtype="bf16", k_dtype="bf16", mode="varlen" if packed else "prefill", seed=460)
    _run(W.pack(wl) if packed else wl, n=48)


@pytest.mark.parametrize("T,H,d,B,m,k", [
    (65, 4, 64, 16, 4, 50), (900, 9, 36, 8, 9, 65), (129, 3, 4, 16, 8, 128), (700, 1, 132, 43, 6, 200), (780, 8, 32, 64, 8, 300),
    (2049, 2, 64, 16, 8, 100), (2100, 5, 32, 17, 9, 130), (1030, 4, 64, 2, 256, 400), (530, 4, 64, 1, 512, 512), (514, 4, 64, 1, 513, 500)])
def test_fp32_rows_in_one_launch(T, H, d, B, m, k):
    # rows around 64, 128, 256 and 512 candidates or blocks (above 512: two launches), heads that are no multiple of
    # four, row pieces that are no 128 bytes; bit for bit against the route that writes its scores, in two launches
    import torch
    from paper_2603_28458_amd import hisa

    wl = W.make_workload(f"rows_f32_{T}", seq_len=T, T=T, H=H, d=d, B=B, m=m, k=k, q_dtype="f32", k_dtype="f32", seed=490)
    print(f"\n[fp32 rows] {wl.name} H={H} d={d} B={B} m={m} k={k}", flush=True)
    Q, K = hisa.to_device(wl)
    Q.w[::7] *= -1.0
    pooled = hisa.hisa_pool_blocks(K, B, pooled_dtype=hisa.HISA_F32)
    blocks = hisa.hisa_block_score_topk(Q, K, pooled, hisa.HISA_F32, B, m)[0]
    assert torch.equal(blocks, hisa.hisa_block_score_topk(Q, K, pooled, hisa.HISA_F32, B, m, want_scores=True)[0])
    ids, sc = hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k, want_topk_scores=True)[:2]
    want, want_sc = hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k, want_topk_scores=True, want_cand_scores=True)[:2]
    assert torch.equal(ids, want) and torch.equal(sc, want_sc)


@pytest.mark.parametrize("T,H,d,M,m,B", [
    (300, 4, 64, 255, 15, 17), (700, 3, 64, 256, 16, 16), (300, 4, 96, 257, 257, 1), (900, 8, 64, 512, 8, 64), (520, 4, 128, 511, 7, 73),
    (300, 1, 64, 64, 8, 8), (2100, 2, 32, 65, 13, 5), (700, 4, 64, 129, 3, 43), (300, 2, 36, 200, 10, 20), (300, 7, 96, 400, 10, 40),
    (700, 3, 132, 100, 5, 20)])
def test_fp32_rows_in_one_launch_with_scores_that_are_no_numbers(T, H, d, M, m, B):
    # rows of M blocks and m * B candidates at the edges of the instances, all in one launch; NaN and infinite scores, -inf
    # (dropped), several sequences, queries that see nothing, part of a block or a later part of a stream: bit for bit as in two
    import torch
    from paper_2603_28458_amd import hisa
    from tests.host_rules import f32_one_launch

    assert f32_one_launch(T, M, H, d) and f32_one_launch(T, m * B, H, d)
    print(f"\n[fp32 rows, specials] T={T} H={H} d={d} M={M} m={m} B={B}", flush=True)
    rng = np.random.default_rng(T + M)
    g = torch.Generator().manual_seed(T)
    n, L, k = 3, M * B, max(1, m * B // 2)
    q, w, keys = torch.randn((T, H, d), generator=g), torch.rand((T, H), generator=g), torch.randn((n, L, d), generator=g)
    w[::5] *= -1.0
    q[3::20, :, 0] = 3e38
    q[4::20, 0, 1] = float("nan")
    w[6::20, 0] = float("inf")
    keys[0, L // 2:: 7, 2], keys[1, L // 3, 0], keys[2, ::3] = float("nan"), float("inf"), keys[2, 0].clone()      # the last: ties
    pooled = torch.randn((n, M, d), generator=g)
    pooled[0, M // 2], pooled[1, M // 3, 0], pooled[2, M // 4: M // 2] = float("nan"), float("inf"), pooled[2, 0].clone()
    lens = np.array([L, max(1, (3 * L) // 4), L - 1])
    seq = rng.integers(0, n, T)
    pos = rng.integers(0, lens[seq])
    pos[::13] = lens[seq[::13]] - 1
    pos[::97] = -1
    lo = np.where(np.arange(T) % 4 == 0, rng.integers(0, np.maximum(1, pos + 1)), 0)
    ints = lambda x: torch.from_numpy(x.astype(np.int32)).cuda()
    Q = hisa.Queries(q=q.cuda(), w=w.cuda(), dtype=hisa.HISA_F32, q_seq=ints(seq), q_pos=ints(pos), q_lo=ints(lo))
    K = hisa.Keys(k=keys.cuda(), seq_len=ints(lens), dtype=hisa.HISA_F32)
    P = pooled.cuda()
    blocks = hisa.hisa_block_score_topk(Q, K, P, hisa.HISA_F32, B, m)[0]
    assert torch.equal(blocks, hisa.hisa_block_score_topk(Q, K, P, hisa.HISA_F32, B, m, want_scores=True)[0])
    ids, sc = hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k, want_topk_scores=True)[:2]
    want, want_sc = hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k, want_topk_scores=True, want_cand_scores=True)[:2]
    assert torch.equal(ids, want) and torch.equal(sc.view(torch.int32), want_sc.view(torch.int32))
    assert torch.equal(hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k)[0], want)


@pytest.mark.parametrize("k_dtype,H,T,B,m", [
    ("bf16", 64, 200, 4096, 2), ("bf16", 32, 130, 1024, 5), ("fp8_e4m3", 64, 255, 512, 9), ("fp8_e4m3", 32, 200, 2048, 3), ("bf16", 64, 3, 4096, 3),
    ("fp8_e4m3", 64, 1, 128, 64), ("bf16", 64, 40, 32, 65), ("bf16", 32, 300, 128, 130),
    ("fp8_e4m3", 32, 1, 32, 7), ("fp8_e4m3", 32, 130, 32, 9), ("fp8_e4m3", 32, 255, 128, 64)])
def test_candidates_in_front_of_and_behind_the_visible_ones(k_dtype, H, T, B, m):
    # large blocks of which a query sees a few tiles, or none, at either end; slots that are empty or name no block, at both ends
    # and between: every candidate's score, -inf where it is masked, against sums in 64 bits
    import torch
    from paper_2603_28458_amd import hisa

    n_blocks = m + 3
    L = n_blocks * B
    print(f"\n[gather] {k_dtype} H={H} T={T} B={B} m={m}", flush=True)
    rng = np.random.default_rng(T + B)
    wl = W.make_workload(f"gather_{T}_{B}", seq_len=L - B // 3, T=T, H=H, d=128, B=B, m=m, k=8, q_dtype="bf16", k_dtype=k_dtype, seed=520)
    pos = rng.integers(0, L, T).astype(np.int32)
    lo = np.where(np.arange(T) % 3 == 0, 0, rng.integers(0, pos + 1)).astype(np.int32)
    lists = np.stack([rng.permutation(np.concatenate([rng.permutation(n_blocks)[: max(1, m - 2)], [-1, n_blocks + 5]]))[:m] for _ in range(T)])
    lists[::4].sort(1)
    lists = np.ascontiguousarray(lists, np.int32)
    Q, K = hisa.to_device(wl)
    Q = hisa.Queries(q=Q.q, w=Q.w, dtype=Q.dtype, q_pos=torch.from_numpy(pos).cuda(), q_lo=torch.from_numpy(lo).cuda())
    got = hisa.hisa_token_refine_topk(Q, K, B, m, torch.from_numpy(lists).cuda(), 8, want_cand_scores=True)[2].cpu().numpy()
    if k_dtype == "bf16":
        keys = K.k[0].double().cpu().numpy()
    else:
        keys = K.k[0].view(torch.float8_e4m3fn).double().cpu().numpy() * K.k_scale[0].double().cpu().numpy()[:, None]
    q, w = Q.q.double().cpu().numpy(), Q.w.double().cpu().numpy()
    n_keys = int(K.seq_len[0])
    for t in range(T):
        tok = (lists[t].astype(np.int64)[:, None] * B + np.arange(B)).reshape(-1)
        seen = np.repeat((lists[t] >= 0) & (lists[t] < n_blocks), B) & (tok <= min(pos[t], n_keys - 1)) & (tok >= lo[t])
        assert np.array_equal(got[t] == -np.inf, ~seen), t
        if t % 16 == 0:
            want = np.maximum(keys[tok[seen]] @ q[t].T, 0.0) @ w[t]
            # fp32 sums of 64 gated heads of 128 products (fp8: the matrix instruction's own accumulation), on the scores' scale
            assert np.abs(got[t][seen] - want).max(initial=0.0) <= (1e-5 if k_dtype == "bf16" else 3e-4) * np.abs(want).max(initial=1.0), t


@pytest.mark.parametrize("k_dtype,H,L,B,m,k", [
    ("bf16", 64, 16500, 32, 200, 700), ("bf16", 64, 17000, 32, 133, 500), ("bf16", 32, 16400, 32, 128, 512), ("bf16", 32, 20000, 64, 120, 900),
    ("fp8_e4m3", 64, 33000, 32, 256, 1000), ("fp8_e4m3", 32, 33000, 32, 100, 400), ("fp8_e4m3", 64, 34000, 128, 128, 2000),
    ("bf16", 32, 16500, 32, 400, 1000)])
def test_walks_that_start_anywhere(k_dtype, H, L, B, m, k):
    # fused Stage 2 over keys that fill more than 4 MB: where a query's walk over its tiles begins follows the clock, and
    # the ids must not: the same bits as the two-kernel route in every call; 4 and 8 waves per query, odd walks,
    # lists with fewer blocks than m (walks of another length), waves with unequal walks
    import time
    import torch
    from paper_2603_28458_amd import hisa

    T = 300
    wl = W.make_workload(f"walk_{k_dtype}_{m}", seq_len=L, T=T, H=H, d=128, B=B, m=m, k=k, q_dtype="bf16", k_dtype=k_dtype, seed=500)
    assert wl.keys.nbytes > 4 << 20
    print(f"\n[walk] {wl.name} H={H} L={L} B={B} k={k}", flush=True)
    Q, K = hisa.to_device(wl)
    rng = np.random.default_rng(501)
    lists = np.sort(np.argsort(rng.random((T, (L - T) // B)), 1)[:, :m], 1).astype(np.int32)
    for t in range(0, T, 3):
        lists[t, int(rng.integers(1, m + 1)):] = -1
    blocks = torch.from_numpy(lists).cuda()
    want = hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k, want_cand_scores=True)[0]
    for i in range(12):
        got = hisa.hisa_token_refine_topk(Q, K, B, m, blocks, k)[0]
        assert torch.equal(got, want), i
        time.sleep(0.0007)
