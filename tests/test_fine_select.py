"""The one-pass top-k (select_topk_fine) on rows it finds hard: scores a few units in the last place apart,
whose bin addresses are rounded coarser than a bin.  Its bin arithmetic (csrc/fine_bins.h) is compiled for the
host and checked there; the kernels that use it are checked on the GPU against a stable sort."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
import torch

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_28458_amd", "csrc")

_SHIM = r"""
#include "fine_bins.h"
static uint32_t cvt(float x) { return !(x >= 0.f) ? 0u : x >= 4294967296.f ? 0xffffffffu : (uint32_t)x; }
static uint32_t med3(uint32_t a, uint32_t lo, uint32_t hi) { return a < lo ? lo : a > hi ? hi : a; }
static uint32_t as_is(uint32_t a, uint32_t, uint32_t) { return a; }
template <int NBIN> void run(const float* x, int n, float lo, float hi, uint32_t base, uint32_t* out, uint32_t* raw) {
  const hisa::FineBins b = hisa::fine_bins<NBIN>(lo, hi, base);
  for (int i = 0; i < n; ++i) {
    out[i] = hisa::fine_bin_address(x[i], b, cvt, med3);
    raw[i] = hisa::fine_bin_address(x[i], b, cvt, as_is);
  }
}
extern "C" void addresses(const float* x, int n, float lo, float hi, uint32_t base, int nbin, uint32_t* out, uint32_t* raw) {
  if (nbin == 2048) run<2048>(x, n, lo, hi, base, out, raw);
  else run<4096>(x, n, lo, hi, base, out, raw);
}
"""


@pytest.fixture(scope="module")
def addresses(tmp_path_factory):
    d = tmp_path_factory.mktemp("fine_bins")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(_SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", str(src), "-o", str(so)], check=True)
    fn = ctypes.CDLL(str(so)).addresses
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_float, ctypes.c_float, ctypes.c_uint32, ctypes.c_int,
                   ctypes.c_void_p, ctypes.c_void_p]

    def call(x, base, nbin):
        x = np.ascontiguousarray(x, dtype=np.float32)
        out, raw = np.empty(x.size, np.uint32), np.empty(x.size, np.uint32)
        fn(x.ctypes.data, x.size, float(np.nanmin(x)), float(np.nanmax(x)), base, nbin, out.ctypes.data, raw.ctypes.data)
        return out.astype(np.int64), raw.astype(np.int64)

    return call


def _ulps_from(start, n):
    """n + 1 consecutive float32 values from `start` away from zero."""
    return (np.float32(start).view(np.uint32) + np.arange(n + 1, dtype=np.uint32)).view(np.float32)


def test_every_score_of_a_narrow_row_has_a_bin(addresses):
    rng = np.random.default_rng(5)
    rows = [_ulps_from(s, n) for s in (3.3, -3.3, 777.7, 1000.0, -1000.0, 1e-30, 1e30) for n in (1, 8, 64, 300, 4000)]
    rows += [_ulps_from(rng.choice([-1, 1]) * 2.0 ** rng.uniform(-100, 100), int(2 ** rng.uniform(0, 16))) for _ in range(300)]
    rows += [np.array(r, np.float32) for r in ([0, 1e-45], [-1e-45, 0, 1e-45], [-1e38, 1e38], [0, 1e38], [1.0, np.nan, 2.0])]
    rows += [np.sort(rng.normal(50, 10, 3000).astype(np.float32))]
    past = 0
    for x in rows:
        for base in (0, 1024, 65536 + 64, 155000 & ~3):
            for nbin in (2048, 4096):
                out, raw = addresses(x, base, nbin)
                top = base + 4 * (nbin - 1)
                assert (out % 4 == 0).all() and out.min() >= base and out.max() <= top, (x[:2], x.size, base)
                order = np.argsort(x, kind="stable")
                order = order[~np.isnan(x[order])]
                assert (np.diff(out[order]) >= 0).all(), (x[:2], x.size, base)
                assert (out[np.isnan(x)] == base).all()
                past += raw.max() > top
    assert past                      # (without the clamp some of these rows leave the bins: it is needed)


# ---------------------------------------------------------------------------------------------------------
def expected_row(scores, ids, k):
    """Top k by (score descending, id ascending), ids ascending, -1 padded; scores / ids of one row."""
    pick = np.sort(ids[np.argsort(-scores, kind="stable")[:k]])
    return np.concatenate([pick, np.full(k - pick.size, -1, pick.dtype)])


def one_head_queries(H, T, weights):
    """T equal queries of H heads of which one is gated: it scores a key by `weights`, {dimension: weight}."""
    from paper_2603_28458_amd import hisa

    q, w = torch.zeros((T, H, 128)), torch.zeros((T, H))
    w[:, 0] = 1.0
    for dim, x in weights.items():
        q[:, 0, dim] = x
    return dict(q=q.bfloat16().cuda(), w=w.cuda(), dtype=hisa.HISA_BF16)


def _rows(dtype, H, T, n_rows, level):
    """Queries that score row r at exactly 1000 + level[r] units in the last place (2^-14): every partial sum
    is a float32 number, so any order of summation gives these scores bit for bit."""
    Q = one_head_queries(H, T, {0: 1.0, 1: 2.0 ** -14, 2: 2.0 ** -6})
    keys = torch.zeros((1, n_rows, 128))
    lv = torch.from_numpy(level)
    if dtype == "bf16":
        keys[0, :, 0], keys[0, :, 1], keys[0, :, 2] = 1000.0, (lv % 256).float(), (lv // 256).float()
        return Q, keys.bfloat16().cuda(), None
    keys[0, :, 0] = 1.0
    scale = (1000.0 + lv.double() * 2.0 ** -14).float()[None]
    return Q, keys.to(torch.float8_e4m3fn).view(torch.uint8).cuda(), scale.cuda()


@pytest.mark.gpu
@pytest.mark.parametrize("spread", [2, 8, 64, 300, 4000])
@pytest.mark.parametrize("dtype,H,m", [("bf16", 64, 128), ("bf16", 32, 128), ("bf16", 64, 250), ("fp8", 32, 128), ("fp8", 32, 250),
                                       ("fp8", 64, 500)])
@pytest.mark.parametrize("T", [40, 300])          # two-kernel and fused Stage 2; the single-launch path too
def test_stage2_on_scores_a_few_ulps_apart(dtype, H, m, T, spread):
    from paper_2603_28458_amd import hisa

    B, k, L = 32, 1000, 16384
    print(f"\n[narrow] {dtype} H={H} m={m} T={T} spread={spread}", flush=True)
    rng = np.random.default_rng(spread)
    level = rng.integers(0, spread, L)
    q, keys, scale = _rows(dtype, H, T, L, level)
    Q = hisa.Queries(**q, q_pos0=L - T - 7)
    K = hisa.Keys(k=keys, seq_len=torch.tensor([L], dtype=torch.int32).cuda(),
                  dtype=hisa.HISA_BF16 if dtype == "bf16" else hisa.HISA_FP8_E4M3, k_scale=scale)
    blocks = np.sort(np.argsort(rng.random((T, L // B)), 1)[:, :m], 1).astype(np.int32)
    got = hisa.hisa_token_refine_topk(Q, K, B, m, torch.from_numpy(blocks).cuda(), k)[0].cpu().numpy()
    pooled = torch.zeros((1, L // B, 128), dtype=torch.bfloat16, device="cuda")
    one_blocks, one, _ = hisa.hisa_indexer_topk(Q, K, pooled, hisa.HISA_BF16, B, m, k, want_block_idx=True)
    one_blocks, one = one_blocks.cpu().numpy(), one.cpu().numpy()
    for t in range(T):
        for lists, ids in ((blocks, got), (one_blocks, one)):
            tok = (lists[t][:, None] * B + np.arange(B)).ravel()
            tok = tok[tok <= L - T - 7 + t]
            assert np.array_equal(ids[t], expected_row(level[tok], tok, k)), t


@pytest.mark.gpu
@pytest.mark.parametrize("spread", [2, 8, 64, 300, 4000])
def test_stage1_on_scores_a_few_ulps_apart(spread):
    from paper_2603_28458_amd import hisa

    B, M, m, T, H = 32, 900, 100, 300, 64      # more than 512 blocks and 256 queries: score rows of their own
    print(f"\n[narrow] stage 1 spread={spread}", flush=True)
    level = np.random.default_rng(spread).integers(0, spread, M)
    q, pooled, _ = _rows("bf16", H, T, M, level)
    Q = hisa.Queries(**q, q_pos0=M * B - T)
    K = hisa.Keys(k=None, seq_len=torch.tensor([M * B], dtype=torch.int32).cuda(), dtype=hisa.HISA_BF16, n_seq=1,
                  s_max=M * B, d=128)
    got = hisa.hisa_block_score_topk(Q, K, pooled, hisa.HISA_BF16, B, m)[0].cpu().numpy()
    for t in range(T):
        own = (M * B - T + t) // B
        ids = np.arange(own + 1)
        score = level[ids].astype(np.float64)
        score[[0, own]] = np.inf                 # forced
        assert np.array_equal(got[t], expected_row(score, ids, m)), t


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["random", "tied", "negative", "nan"])
@pytest.mark.parametrize("M,m", [(40, 3), (70, 69), (300, 126), (512, 2), (1024, 100), (1025, 7), (2048, 64), (2049, 128), (8192, 1000)])
def test_stage1_of_a_small_batch_against_a_sort(M, m, kind):
    # the one-launch Stage 1: queries that see from m + 1 blocks to all of them, some from the middle of a stream on.
    # tied: ties across the threshold and bins crowded by copies of one score.  negative: scores of -inf, which are no candidates.
    # nan: declined; a NaN that comes of an infinite dot product and a gate of 0 has its sign bit set and is the lowest
    # candidate there is, which a query takes, first ids first, when it runs out of others; in blocks that a query does not
    # see it changes nothing.  (A NaN in a key is none in its score: the ReLU makes 0 of it.)
    from paper_2603_28458_amd import hisa

    B, T, H = 32, 24, 64 if M % 2 == 0 else 32
    print(f"\n[small stage 1] M={M} m={m} H={H} {kind}", flush=True)
    rng = np.random.default_rng(M + m)
    level = rng.integers(0, 5, M) if kind == "tied" else rng.permutation(M)
    sign = -1.0 if kind == "negative" else 1.0
    q = one_head_queries(H, T, {0: 1.0, 1: 256.0, 2: 256.0})
    q["w"] *= sign
    pooled = torch.zeros((1, M, 128))
    pooled[0, :, 0], pooled[0, :, 1] = torch.from_numpy(level % 256).float(), torch.from_numpy(level // 256).float()
    score = sign * level.astype(np.float64)
    if kind == "negative":
        gone = rng.permutation(M)[: M // 5]
        pooled[0, gone, 2] = 3e38
        score[gone] = -np.inf
    if kind == "nan":
        q["q"][:, 1, 3] = 3e38
        gone = rng.permutation(M)[: M * 2 // 3]
        pooled[0, gone, 3] = 3e38
        score[gone] = -1e300
    pos = np.sort(np.concatenate([[m * B, m * B + 40, M * B - 1], rng.integers(m * B, M * B, T - 3)])).clip(max=M * B - 1)
    lo = np.where(np.arange(T) % 3 == 0, 0, rng.integers(0, np.maximum(1, pos - m * B)))
    Q = hisa.Queries(**q, q_pos=torch.from_numpy(pos.astype(np.int32)).cuda(), q_lo=torch.from_numpy(lo.astype(np.int32)).cuda())
    K = hisa.Keys(k=None, seq_len=torch.tensor([M * B], dtype=torch.int32).cuda(), dtype=hisa.HISA_BF16, n_seq=1, s_max=M * B, d=128)
    pooled = pooled.bfloat16().cuda()
    got = hisa.hisa_block_score_topk(Q, K, pooled, hisa.HISA_BF16, B, m)[0].cpu().numpy()
    if kind == "nan":
        want, scores = hisa.hisa_block_score_topk(Q, K, pooled, hisa.HISA_BF16, B, m, want_scores=True)
        first = lo[-1] // B                      # (the last query sees every block from there on)
        assert torch.isnan(scores[-1, first:]).sum() == (gone >= first).sum() > 0
        assert np.array_equal(got, want.cpu().numpy())
    for t in range(T):
        ids = np.arange(lo[t] // B, pos[t] // B + 1)
        s = score[ids].copy()
        s[[0, -1]] = np.inf                      # forced
        ids, s = ids[s > -np.inf], s[s > -np.inf]
        assert np.array_equal(got[t], expected_row(s, ids, m)), t


@pytest.mark.gpu
@pytest.mark.parametrize("copies", [2, 20, 64, 65, 300])
@pytest.mark.parametrize("M,m", [(70, 9), (300, 126), (512, 30), (1024, 64), (1025, 7), (2048, 500), (2049, 128), (8192, 1000)])
def test_stage1_of_a_small_batch_with_ties_across_the_threshold(M, m, copies):
    # the one-pass top-m takes the first of the blocks that share the threshold's score, also if they crowd their bin alone (more
    # than 64); with others among them it declines.  Every instance of the one-launch Stage 1, copies side by side, strewn over
    # the row, and strewn with a quarter of them a hair above the rest
    from paper_2603_28458_amd import hisa

    B, T, H = 32, 24, 64 if M % 2 == 0 else 32
    print(f"\n[small stage 1, ties] M={M} m={m} H={H} copies={copies}", flush=True)
    rng = np.random.default_rng(M + m + copies)
    K = hisa.Keys(k=None, seq_len=torch.tensor([M * B], dtype=torch.int32).cuda(), dtype=hisa.HISA_BF16, n_seq=1, s_max=M * B, d=128)
    strewn = rng.permutation(M) // copies
    beside = strewn.astype(np.float64)
    beside[rng.permutation(M)[: M // 4]] += 2.0 ** -12              # in the bin of the others; every sum below is a float32 number
    for level in (rng.permutation(-(-M // copies)).repeat(copies)[:M], strewn, beside):
        pooled = torch.zeros((1, M, 128))
        pooled[0, :, 0], pooled[0, :, 1] = torch.from_numpy(level // 1 % 256).float(), torch.from_numpy(level // 256).float()
        pooled[0, :, 2] = torch.from_numpy(level % 1).float()
        pos = np.concatenate([rng.integers(m * B, M * B, T - 1), [M * B - 1]])
        lo = np.where(np.arange(T) % 3 == 0, rng.integers(0, np.maximum(1, pos - m * B)), 0)
        Q = hisa.Queries(**one_head_queries(H, T, {0: 1.0, 1: 256.0, 2: 1.0}), q_pos=torch.from_numpy(pos.astype(np.int32)).cuda(),
                         q_lo=torch.from_numpy(lo.astype(np.int32)).cuda())
        got = hisa.hisa_block_score_topk(Q, K, pooled.bfloat16().cuda(), hisa.HISA_BF16, B, m)[0].cpu().numpy()
        for t in range(T):
            ids = np.arange(lo[t] // B, pos[t] // B + 1)
            s = level[ids].astype(np.float64)
            s[[0, -1]] = np.inf                      # forced
            assert np.array_equal(got[t], expected_row(s, ids, m)), t


@pytest.mark.gpu
@pytest.mark.parametrize("T,H,M,m", [(257, 64, 512, 64), (1024, 64, 511, 500), (1025, 64, 512, 64), (300, 64, 33, 2), (700, 64, 130, 32),
                                     (1536, 32, 512, 128), (1537, 32, 512, 64), (769, 32, 64, 63), (258, 32, 3, 2), (600, 32, 513, 64)])
def test_stage1_in_one_launch_beyond_a_query_per_cu(T, H, M, m):
    # edges of the rule and of the tiles, bit for bit against the route that writes its scores (two kernels): ragged
    # sequences, queries that see nothing, all they can or a later part of a stream, ties, scores of -inf and +inf, NaN
    from paper_2603_28458_amd import hisa

    B, n = 32, 3
    print(f"\n[stage 1, one launch] T={T} H={H} M={M} m={m}", flush=True)
    rng = np.random.default_rng(T + M)
    g = torch.Generator().manual_seed(T)
    q = torch.randn((T, H, 128), generator=g).bfloat16()
    w = torch.rand((T, H), generator=g)
    w[::11] *= -1.0
    pooled = torch.randn((n, M, 128), generator=g)
    pooled[0, M // 3: M // 2] = pooled[0, M // 3].clone()           # ties
    q[5::50, :, 0] = 3e38                                           # infinite scores
    q[7::50, :, 1] = float("nan")
    if M <= 512:
        pooled[2, M // 2] = float("nan")
    seq = rng.integers(0, n, T)
    lens = np.array([M * B, max(1, (M * B * 3) // 4 - 5), M * B - 1])
    pos = rng.integers(0, lens[seq])
    pos[::13] = lens[seq[::13]] - 1
    pos[::97] = -1
    lo = np.where(np.arange(T) % 4 == 0, rng.integers(0, np.maximum(1, pos + 1)), 0)
    ints = lambda x: torch.from_numpy(x.astype(np.int32)).cuda()
    K = hisa.Keys(k=None, seq_len=ints(lens), dtype=hisa.HISA_BF16, n_seq=n, s_max=M * B, d=128)
    P = pooled.bfloat16().cuda()
    Q = hisa.Queries(q=q.cuda(), w=w.cuda(), dtype=hisa.HISA_BF16, q_seq=ints(seq), q_pos=ints(pos), q_lo=ints(lo))
    K1 = hisa.Keys(k=None, seq_len=ints(lens[:1]), dtype=hisa.HISA_BF16, n_seq=1, s_max=M * B, d=128)
    C = hisa.Queries(q=q.cuda(), w=w.cuda(), dtype=hisa.HISA_BF16, q_pos0=max(0, M * B - T))   # consecutive
    for queries, keys, pk in ((Q, K, P), (C, K1, P[:1].contiguous())):
        got = hisa.hisa_block_score_topk(queries, keys, pk, hisa.HISA_BF16, B, m)[0]
        want = hisa.hisa_block_score_topk(queries, keys, pk, hisa.HISA_BF16, B, m, want_scores=True)[0]
        bad = (got != want).any(1).nonzero().flatten()
        assert bad.numel() == 0, (bad[:8].tolist(), got[bad[0]].tolist(), want[bad[0]].tolist())
