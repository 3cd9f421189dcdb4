// Launch rules of the linear kernels: which variant, k-ranges, tiles and grid a pass takes, as plain host
// functions of sizes and types, so that they can be checked over every accepted shape without a GPU.
#pragma once
#include <algorithm>
#include <cstddef>

namespace seedk {

enum Epilogue { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_HEAD = 3 };

// LDS of a CU, all of which one workgroup may take (seed_create refuses a device that grants less)
constexpr size_t LDS_MAX = 160 * 1024;
constexpr int ACT_TILE = 2048;      // bytes of a packed activation tile (layout in kernels.h)

constexpr int ROWS_HEAD_NT = 2;     // n-tiles per argmax partial of a small vocabulary's head (rows.hip)
constexpr int ROWS_KS_MAX = 16;     // k-ranges of a decode pass's projection
constexpr int ROWS_THREADS = 512;   // largest workgroup of k_linear_rows (its launch bounds),
constexpr int ROWS_PART_THREADS = 128;   // of the form whose k-ranges go to several workgroups
constexpr size_t ROWS_LDS = 150 * 1024;   // partial sums of one workgroup (its row scales take 256 bytes more)

inline size_t rows_lds(int NT, int KS, int M) { return (size_t)NT * KS * M * 16 * sizeof(float); }

// K-ranges, a function of the weight shape only: 8 where N gives the chip enough workgroups (QKV, gate/up)
// and for a small vocabulary's head; else ranges of about 16 k-tiles, at most 8, the waves of one workgroup.
// Only the residual projections have a form with more (16: rows_plan's part).
inline int rows_ks(int n_tiles, int KT, int epilogue) {
  if (n_tiles >= 256 || epilogue == EPI_HEAD) return std::min(8, KT);
  return std::min(epilogue == EPI_RESID ? ROWS_KS_MAX : ROWS_THREADS / 64, std::max(1, KT / 16));
}

// n-tiles per workgroup: the fewest rounds of one workgroup per CU x (n-tiles + half a tile's time to
// start), among those whose partial sums fit LDS (5 only up to 48 rows: its sums and operands fill the
// registers). Measured at 5 rows, us for NT = 1 / 2 / 3 / 5: gate/up of the 4B shape (1216 n-tiles) 19.9 /
// 20.9 / 20.0 / 17.9, QKV (384) 10.3 / 9.0 / 10.7 / 13.2, O (160) 8.2 / 10.4 / 12.4 / 16.6; at 8 rows gate/up of
// the 28-layer shape (768) 16.9 / 15.6 / 11.9 / 13.5.
inline int rows_nt(int n_tiles, int KS, int M) {
  const int cands[] = {5, 3, 2, 1};
  int best = 1;
  long long best_cost = -1;
  for (int nt : cands) {
    if (rows_lds(nt, KS, M) > ROWS_LDS || (nt == 5 && M > 48)) continue;
    const long long cost = (((n_tiles + nt - 1) / nt + 255) / 256) * (2 * nt + 1);
    if (best_cost < 0 || cost < best_cost) best = nt, best_cost = cost;
  }
  return best;
}

// A decode pass's projection (M <= 64 rows, N x K weights of esize bytes): its k-ranges, n-tiles per
// workgroup and grid. part: the k-ranges go to several workgroups, two each, and a second kernel adds them.
struct RowsPlan {
  int KS, NT;
  bool part;
  int gx, gy, threads;
  size_t lds;
};

inline RowsPlan rows_plan(int N, int K, int M, int epilogue, int esize) {
  const int n_tiles = N >> 4;
  RowsPlan p;
  p.KS = rows_ks(n_tiles, K >> 5, epilogue);
  // More than 8 k-ranges (a long K into a narrow N: the down projection): two ranges per workgroup, NT n-tiles
  // each, and a reduction. All ranges in one workgroup would give 160 workgroups at the 4B shape, each
  // reading every row's activations: 15.2 us at 5 rows and 31.5 at 40, against 10.2 + 4.5 and 14.0 + 5.1. Fewer rows gain
  // nothing from it either: verification of 2 rows (36 layers) 2.141 ms as it is, 2.173 in one launch; a draft
  // step 235 and 237 us.
  p.part = epilogue == EPI_RESID && p.KS > 8;
  if (p.part)
    // 5 n-tiles where that still makes about two waves per CU, else 2 (28-layer down, 128 x 12 ranges, 31
    // rows: 11.0 us with 2, 11.7 with 3; 4B down, 160 x 16, 40 rows: 22.4 / 17.0 / 14.0 with 2 / 3 / 5)
    p.NT = esize == 2 && (n_tiles + 4) / 5 * p.KS >= 480 ? 5 : 2;
  else if (epilogue == EPI_HEAD)
    p.NT = ROWS_HEAD_NT;
  else
    // fp32 operands take twice the registers: 1 n-tile, 2 k-tiles in flight (launch_rows_tt), not tuned further.
    // Against the kernels that staged rows in LDS, verification of two 4B layers in fp32, whole calls at 1 / 5 / 16 / 17 /
    // 40 / 64 rows: 358 / 366 / 410 / 493 / 682 / 930 -> 245 / 276 / 341 / 353 / 465 / 572 us (about 55 of it outside the
    // kernels); four steps of two 28-layer shapes' layers for 8 sequences 955 -> 716.
    p.NT = esize == 4 ? 1 : rows_nt(n_tiles, p.KS, M);
  p.gx = (n_tiles + p.NT - 1) / p.NT;
  p.gy = p.part ? (p.KS + 1) / 2 : 1;
  p.threads = p.part ? ROWS_PART_THREADS : 64 * p.KS;
  p.lds = p.part ? 0 : rows_lds(p.NT, p.KS, M);
  return p;
}

// ---- LM head of a decode pass ----
constexpr int HEAD_NT = 8;   // n-tiles per argmax partial of the head's own kernels (waves of a workgroup)
constexpr int HEAD_CK = 8;   // k-tiles per chunk that k_head_chunked stages

// Small vocabularies split K over waves like the other projections: at 1024 tokens the head's kernels would have 8
// workgroups, each wave a chain over all of K (5 rows 19 us, 40 rows 55). The line is on the safe side of that,
// not where the two meet: a verification with one thin layer of hidden size 2560 takes, at 1 / 5 / 17 / 40 / 64 rows, 87 / 95 /
// 114 / 152 / 187 us with 32000 tokens (row kernel) and 84 / 92 / 96 / 118 / 139 with 32768 (head's kernels).
inline bool head_by_rows(int N) { return N < 32768; }
// n-tiles per argmax partial
inline int head_group(int N) { return head_by_rows(N) ? ROWS_HEAD_NT : HEAD_NT; }

// k_head_lds stages all rows (M <= 16): 32 bytes per row and 8 features, one zero slot, the sums and row scales
inline size_t head_lds_bytes(int M, int K) {
  return (size_t)(K >> 5) * 4 * M * 32 + 32 + (size_t)(HEAD_NT * M + 1) * 16 * sizeof(float);
}

struct HeadPlan {
  bool chunked;   // k_head_chunked, NT n-tiles per wave; else k_head_lds
  int NT, grid;
  size_t lds;
};

inline HeadPlan head_plan(int N, int K, int M, int esize) {
  const int n_tiles = N >> 4;
  if (M <= 16 && head_lds_bytes(M, K) <= LDS_MAX)
    return {false, 1, (n_tiles + HEAD_NT - 1) / HEAD_NT, head_lds_bytes(M, K)};
  // 5 n-tiles per wave (the largest whose sums and operands fit the registers of two waves per SIMD) from the
  // vocabulary on that makes half a round of workgroups of them, one per CU. At 151936 tokens, one round, 31 rows of the
  // 28-layer shape take 120 us against 146 with 16 waves of one n-tile. At the line itself one n-tile is
  // still the faster: a verification with one thin layer of hidden size 2560 at 17 / 31 / 40 / 64 rows takes 143 / 153 / 190 / 225 us with
  // 81904 tokens (1 n-tile) and 162 / 176 / 195 / 229 with 81920 (5).
  const int nt = esize == 2 && n_tiles >= 128 * 5 * HEAD_NT ? 5 : 1, per = nt * HEAD_NT;
  return {true, nt, (n_tiles + per - 1) / per, 2 * (size_t)((M + 15) / 16) * HEAD_CK * ACT_TILE};
}

// ---- wide passes ----
constexpr int WIDE_MJ = 4;   // token tiles per workgroup (64 rows)

// K-ranges of the residual projections: 2 for N <= 4096, whose workgroups do not fill the chip otherwise (1024
// rows x 2560: 128 of 20 n-tiles); a function of the weight shape only, so that a row's output does not depend
// on the pass's row count.
constexpr int WIDE_SPLIT_MAX = 2;   // (partials: WIDE_SPLIT_MAX x rows x N floats)
inline int wide_split(int n_tiles, int KT) { return std::max(1, std::min(n_tiles <= 256 ? WIDE_SPLIT_MAX : 1, KT / 4)); }

// n-tiles per wave: the candidate with the lowest rounds of one workgroup per CU x (n-tiles + a fixed
// part for the token tiles' staging, which every n-tile of the wave shares), a quarter more when there
// is one round only (a lone workgroup on a CU has none to overlap its barriers). Measured, us for NI =
// 3 / 4 / 5 / 6: gate/up (1216 n-tiles) of 1024 rows 189 / 170 / 166 / 183, of 4096 rows NI = 4 / 5 / 6
// 716 / 678 / 669; QKV (384) of 1024 rows 65 / 78 / 88 / 65; O and down (160 in 2 k-ranges, mean) 77 / 91
// / 63 / 70. 8 token tiles per workgroup instead of 4 (one wave per SIMD) were slower at every width
// (prefill of 4 layers 2.92 against 2.26 ms).
inline int wide_ni(int n_tiles, int M, int S) {
  const int MT = (((M + 15) >> 4) + WIDE_MJ - 1) / WIDE_MJ;
  int best = 0;
  long long best_cost = -1;
  for (int ni = 6; ni >= 1; --ni) {
    const long long wgs = (long long)((n_tiles + 4 * ni - 1) / (4 * ni)) * MT * S;
    const long long rounds = (wgs + 255) / 256, cost = rounds * (10 * ni + 12) * (rounds == 1 ? 5 : 4);
    if (best_cost < 0 || cost < best_cost) best = ni, best_cost = cost;
  }
  return best;
}

// ---- attention of decode passes ----
// Positions per attention group for a context capacity and batch capacity (fixed per decoder, so
// that a query's merge tree depends only on absolute positions).
// One sequence: 64 positions per group up to 4096 (at its ~1.2k-position context, 1024-token
// prompt, 128-position groups leave half the 160 workgroups of a launch out: verification
// attention 7.9 -> 9.6 us per layer). Several sequences fill the chip sooner: 64 while max_batch (8 at
// most) x positions stay within 8192, and up to 2048, then 128 (8 ragged sequences of up to 2048 positions:
// verification attention 18.4 -> 16.2 us per layer and its merge 9.2 -> 7.2 us against 64; at ~2300 positions
// 19.7 -> 17.4, 256 gave 19.3). 256 beyond 8192 positions (16k contexts).
inline int attention_span(int max_ctx, int max_batch) {
  const int small = max_batch == 1 ? 4096 : std::min(2048, 8192 / std::min(max_batch, 8));
  return max_ctx <= small ? 64 : (max_ctx <= 8192 ? 128 : 256);
}

}  // namespace seedk
