"""Parity at the edges of the size-dependent dispatch rules: each case sits where one kernel hands over
to another, or where the way a kernel divides its work changes."""
import numpy as np
import pytest

from paper_2603_28458_amd import workloads as W
from tests.parity import run_and_check, sample_queries

pytestmark = pytest.mark.gpu


def _run(wl, n=24, **kw):
    print(f"\n[parity] {wl.name}: T={wl.T} H={wl.H} B={wl.B} m={wl.m} k={wl.k} k={wl.k_dtype} n_seq={wl.n_seq} "
          f"s_max={wl.s_max} seed={wl.seed}", flush=True)
    return run_and_check(wl, queries=sample_queries(wl, n), **kw)


@pytest.mark.parametrize("T,L,k_dtype", [(64, 9001, "bf16"), (71, 4097, "fp8_e4m3"), (257, 30000, "bf16"),
                                         (1000, 6400, "fp8_e4m3"), (2055, 2055, "bf16")])
def test_key_ranges_of_the_prefill_scoring_kernel(T, L, k_dtype):
    # the dense scoring kernel (flat indexer, Stage 1 of a chunk) cuts the keys of 8 queries into ranges of
    # 128-key tiles: 9, 8, 2 and 1 queries groups over the CUs, uneven ranges, ranges past a short prefix
    wl = W.make_workload(f"ranges{T}", seq_len=L, T=T, H=64, d=128, B=32, m=20, k=512, q_dtype="bf16",
                         k_dtype=k_dtype, seed=400 + T)
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
