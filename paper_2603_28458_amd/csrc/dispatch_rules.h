// How a launch's work is cut into workgroups, from its sizes alone: plain arithmetic, so that a host compiler
// can take the same lines.
#pragma once

namespace hisa {

constexpr int kCUs = 256;
constexpr long kLdsPerCU = 160 * 1024;

// Workgroups per 8 queries of k_score_prefill: the key tiles (128 rows) of 8 queries are cut into that many
// ranges.  rows_first, rows_last: what the first and the last query see; the queries between them grow evenly and
// the longest start first.  A CU holds one workgroup.  With a workgroup's time as its tiles and three more, the
// launch takes at least as long as its longest workgroup, as its work spread over the CUs, and as r times its
// 256 (r - 1) + 1-th longest when there are r rounds (a CU has r of them at least that long); this takes the
// fewest ranges within 2 % of the least.  1024 queries at 64K keys: 128 workgroups, 1497 us with the select; 256
// (split by 2) 964 us; 512 queries 1369 -> 494 us (by 4), 100 queries at 128K fp8 keys 2605 -> 340 us (by 16).
// Over 416 calls (64 to 16000 queries, 300 to 200000 rows, flat and Stage 1), measured with 1 .. 32 ranges, the
// rule is 0.2 % from the best on average and 6 % at most, and one is 3 % slower than unsplit.  (Priced by the length
// of the key array and as if every query saw all of it: 3000 queries of a 4000-key prefill 5 % slower than
// unsplit, 1500 queries at 300 of 4096 blocks 33 -> 44 us.)  From four rounds on the split is left alone: 8 rounds
// of 16K-key rows measured the same with 1, 2 and 4.
inline int prefill_split(long q_groups, long rows_first, long rows_last) {
  if (q_groups >= 4 * kCUs) return 1;
  const double hi = (double)((rows_last + 127) / 128), lo = rows_first < 128 ? 1.0 : rows_first / 128.0;
  int best = 1;
  double best_cost = 0.0;
  for (int s = 1; s <= 32 && (s == 1 || s <= hi); ++s) {
    const long wgs = q_groups * s, rounds = (wgs + kCUs - 1) / kCUs;
    const double longest = hi / s + 3.0;
    const double work = (wgs * 3.0 + q_groups * (hi + lo) / 2.0) / kCUs;
    const double last_round = rounds * ((hi - (hi - lo) * (double)(kCUs * (rounds - 1)) / wgs) / s + 3.0);
    double cost = longest > work ? longest : work;
    cost = cost > last_round ? cost : last_round;
    if (s == 1 || cost < best_cost * 0.98) {
      best_cost = cost;
      best = s;
    }
  }
  return best;
}

// Tiles per wave of k_score_gather (Stage 2 of a decode batch).  A workgroup's four waves
// walk tpw tiles each behind a set-up (query, position, block list) worth about six tiles.  Two workgroups on
// a CU take twice as long as their share of it, one alone three quarters of that (nothing covers its waits):
// a full round of 2 * kCUs workgroups counts 4, a last round 4 or, with at most one per CU, 3.
// One wave per tile keeps a single query's latency short, a wide batch wants full rounds of long workgroups.
// Refinement calls, us at the value picked here (in brackets at 4), B 128: bf16 keys, 64 heads: 1 query, m 64 1: 10.3 (11.9);
// 32, m 64 4: 21.0; 77, m 32 6: 22.3 (23.9); 130, m 64 10: 52.9 (53.2); 200, m 32 16: 39.3 (43.4); 200, m 64 13: 88.6 (90.9);
// 255, m 128 16: 221.5 (217.4); fp8 keys: 32, m 64 4: 16.6; 130, m 32 11: 21.1 (27.3); 200, m 64 13: 44.9 (50.8).  Over 140 such
// calls (1 to 255 queries, 16 to 512 tiles, both key types, 32 and 64 heads) the rule is 1.1 % from the best of 1 .. 16 on average
// and 12 % at most (255 queries of 64 tiles, fp8); against 4 tiles it is 6 % faster on average and 5 % slower at
// most.
inline int gather_tiles_per_wave(long T, long n_tiles) {
  int best = 1;
  long best_cost = 0;
  for (int tpw = 1; tpw <= 16; ++tpw) {
    const long wgs = T * ((n_tiles + 4 * tpw - 1) / (4 * tpw));
    const long rest = wgs % (2 * kCUs);
    const long cost = (4 * (wgs / (2 * kCUs)) + (rest > kCUs ? 4 : rest > 0 ? 3 : 0)) * (tpw + 6);
    if (tpw == 1 || cost < best_cost) {
      best_cost = cost;
      best = tpw;
    }
  }
  return best;
}

// Waves per query of k_rows_f32 (fp32 rows of at most 512 candidates, 64 of which a wave scores at a time; a workgroup
// holds 9 KB of LDS per wave).  Few queries: a wave for every 64 candidates, so that none scores twice in a row.  Many:
// half as many, since a wave that only waits for the others' scores keeps its LDS.  Refinement, us with 1 / 2 / 4 / 8
// waves (two launches: the last figure): 300 queries of 512 candidates 28.6 / 21.1 / 17.4 / 13.4 (16.3), 600 of 512
// 43.7 / 28.7 / 22.2 / 19.7 (23.3), 1024 of 256 20.4 / 15.1 / 12.8 / 18.7 (18.6), 1500 of 96 14.6 / 12.3 / 18.5 (21.0),
// 3000 of 512 43.4 / 44.6 / 46.9 / 64.6 (53.8); Stage 1: 2000 of 125 blocks 10.3 / 9.3 / 13.6 (15.3), 3000 of 94
// 19.3 / 21.3 / 29.9 (20.9), 3000 of 47 10.6 / 15.0 / 20.6 (14.7).
inline int rows_f32_waves(long T, long n_max) {
  const long per_wave = T > 2048 ? 128 : 64;
  const int nw = n_max <= per_wave ? 1 : n_max <= 2 * per_wave ? 2 : n_max <= 4 * per_wave ? 4 : 8;
  return nw == 8 && T > 768 ? 4 : nw;
}

// fp32 rows of at most 512 candidates: scored and selected in one launch (k_rows_f32), or in two (k_score_ranges_f32 and
// the select)?  T queries, n_max candidates, H heads of d elements.  In one launch a launch is saved and the key rows come
// in whole pieces of 128 bytes, 4 heads at a time; but a wave takes such a step (4 heads, 8 chunks of 16 bytes) in 1 us
// however few of the 8 chunks a row has, 64 candidates have one wave, and a workgroup keeps 9 KB of LDS per wave until its
// first wave has selected.  In two, a row is cut over all CUs and costs d / 4 shorter steps, heads beyond a multiple of four
// one at a time.  Both are priced, in us: launches, the longest chain of one workgroup (a second round of workgroups
// follows two thirds of a first one later) and what all of them take from a CU.  The prices hold to a few percent for a few heads
// of whole pieces and to 10-20 % elsewhere, where one launch has to be 10 % better.  us in one launch (in two): 1024 queries of 256, 4
// heads of 64: 13.4 (17.3); 700 of 512, 4 of 64: 18.3 (21.4); 3000 of 512, 4 of 4: 28 (17.4); 6000 of 32, 128 of 16: 485 (64);
// 1024 of 64, 64 of 128: 122 (77); 2048 of 512, 16 of 128: 135 (237), 3 of 512: 182 (1488); 100 of 512, 128 of 32: 45 (66).
// Over 45768 calls (1 to 16000 queries, 20 to 512 candidates, 1 to 128 heads of 4 to 512, both stages) the rule is 1.8 %
// from the better one on average; what it takes in one launch is at most 5 % slower there in 95 of 100 calls and 16 % in 99
// (everything in one launch: up to 7.6 times slower).
inline bool rows_f32_one_launch(long T, long n_max, int H, int d) {
  const int pieces = d / 4, whole = pieces / 8, rest = pieces % 8;
  const double four_heads = whole + (rest ? 0.6 + 0.1 * rest : 0.0);
  const double fewer_heads = 0.6 * ((pieces + 7) / 8) + 0.1 * pieces;
  const double step = H / 4 * four_heads + (H % 4 ? fewer_heads : 0.0);
  const long waves = rows_f32_waves(T, n_max), tasks = (n_max + 63) / 64, passes = (tasks + waves - 1) / waves;
  const long rounds = (T * waves + 16 * kCUs - 1) / (16 * kCUs);   // 16 waves' LDS on a CU
  const double one = (passes * step + 7.5) * (1.0 + 0.67 * (rounds - 1)) + T * tasks * step / 3000.0;
  const double row = pieces * (H / 4 * 0.065 + H % 4 * 0.095);
  const double two = 9.0 + row * ((n_max + 255) / 256 + T * tasks / 1400.0) + 0.0012 * T +
                     7e-7 * T * n_max * ((H + 3) / 4) * pieces;
  return one < (rest == 0 && H * d <= 1024 ? 1.05 : 0.9) * two;
}

// Stage 1 in one launch (k_stage1_query), or scoring and select in two?  T queries of M blocks, H heads.
// Up to a query per CU, any row that the select holds.  Beyond, workgroups of 4 waves, of which a
// CU holds two (64 heads, by registers) or three (32, by LDS); each round of them takes 6-9 us, and the two launches,
// which are better at many queries, 9-16 us at first.  us in one launch (in two: queries with positions of their
// own / consecutive), 512 blocks, 64 heads: 257 queries 8.4 (11.7 / 14.6), 512 8.9 (12.4 / 16.4), 640 13.5 (15.9 / 17.6), 1024
// 16.0 (17.5 / 19.4), 1300 22.5 (22.4 / 22.6), 2047 31.3 (30.2 / 26.2); 32 heads: 768 9.1 (14.3 / 14.2), 1024 13.8 (15.8 /
// 14.6), 1536 15.9 (19.7 / 18.0), 2047 21.6 (23.7 / 18.5); 128 blocks, 64 heads: 512 6.8 (10.1 / 14.8), 1024 12.0 (13.3 / 15.9),
// 1300 16.7 (16.0 / 16.4).  So: two rounds.  Over 512 blocks the two launches' select is another one,
// with workgroups of its own for a row, and one launch is not measured against it.
inline bool stage1_one_launch(long T, long M, int H) {
  return T <= kCUs ? M <= 8192 : M <= 512 && T <= 2 * kCUs * (H == 64 ? 2 : 3);
}

// Workgroups that a CU holds: by their LDS, and at most max_wgs of them by their registers.
inline int wgs_per_cu(long lds, int max_wgs) {
  const long n = kLdsPerCU / lds;
  return n < 1 ? 1 : n < max_wgs ? (int)n : max_wgs;
}

// Fused Stage 2: ticks (10 ns) that a wave takes for two tiles of 32 keys, by which the walks of all workgroups are laid
// over each other (k_refine_fused); 0 where the key array of a sequence fits an XCD's L2 anyway.  What they take depends on how
// often the tiles miss the L2, so on the ticks themselves.  us of a launch, two cards within 1 %, m 64 unless stated:
//   bf16 keys                       no walk   140   160   180   200   220   240   280 ticks
//   64 heads, 20000 at 128K           4094   3354  2799  2794  2857  2922  2944  3025
//             16000 at 256K           3824   3686  3471  3193  2617  2682  2763  2894
//             8000 at 500K            1987   1956  1888  1806  1762  1731  1731  1730
//             prefill of 64K          8247   7954  7974  8004  7980  8016  8051  8053
//             16000 at 256K, m 128    7515   7323  6446  5643  5171  5209  5284  5463
//   32 heads, 20000 at 128K           4284   2415  2414  2508  2604  2746  2904  3032
//             16000 at 256K           3885   3856  3568  3373  3163  3107  3114  3044
//   fp8 keys                        no walk   110   130   145   160   175   200   230 ticks
//   64 heads, 20000 at 256K           2326   2315  2282  2296  2300  2295  2315  2332
//             16384 at 1M, m 128      4283   4209  4170  4161  4173  4151  4181  4192
//   32 heads, 12000 at 128K            970    874   861   855   895   884   905   904
//             16000 at 500K           1939   1880  1760  1677  1426  1453  1503  1550
//             16384 at 500K, m 128    3740   3125  3142  3199  3228  3252  3290  3349
// Too long costs little, too short a lot: 10 % below these two values 16000 queries at 256K and at 500K lose 22 and 17 %, 10 % above
// 2 %; so a card that is 10 % slower would lose that (no value in the table is slower than no walk by more than it is uncertain,
// 0.5 %).  32 heads share the durations: they wait for the same tiles.
// By the length of the key array, not by what the queries see (which the host need not know): queries that see little of a
// long array walk for nothing, and lose nothing by it: prefills of 9000 to 20000 tokens in an array of 128K 622 to 2029 us
// (624 to 2027 without), 8 sequences of 16000 tokens in arrays of 64K 2059 (2057), 32 of 12000 1652 (1654), fp8 keys, 8 of
// 30000 1700 (1692), 24K packed prefill 411 (408).
inline unsigned walk_ticks(long key_bytes, bool fp8) {
  return key_bytes <= 4l << 20 ? 0u : fp8 ? 160u : 200u;
}

// Fused Stage 2 with 32 heads: do the top-k's bins lie in the tile rings, so that `with` instead of `without`
// workgroups fit on a CU (k_refine_fused, wgs_per_cu)?  One more workgroup hides more of the tiles' latency (16K prefill,
// m 32, bf16 keys 733 -> 668 us, fp8 keys, m 64 +10 %), except where
// * it saves no round over the CUs: the same rounds are then only longer (fp8 keys, m 64, 2 -> 3 workgroups:
//   600 queries 28 % faster, 1000 queries 7 % slower; m 32, 3 -> 4: 1000 queries 24 % faster, 1200 3 % slower);
// * three workgroups' tiles wash each other out of the 4 MB L2 of their XCD: bf16 keys of 64K tokens of one
//   sequence, queries that agree on nothing, 1058 -> 1294 us (neighbours that agree: 972 -> 865).  Up to 48K tokens
//   every measured call gains 4-13 %, at 56K some lose up to 13 %, at 64K 18 %.  The queries of a packed stream see
//   only a part of it (pieces of 4K to 48K of a 64K or 128K stream gain 8-15 %; one piece of 64K loses 4 %);
//   fp8 keys are half as wide (64K: +10 to 18 %).
inline bool hist_in_ring(long T, long s_max, bool packed, bool fp8, int without, int with) {
  if ((T + kCUs * with - 1) / (kCUs * with) >= (T + kCUs * without - 1) / (kCUs * without)) return false;
  return fp8 || packed || s_max <= 49152;
}

}  // namespace hisa
