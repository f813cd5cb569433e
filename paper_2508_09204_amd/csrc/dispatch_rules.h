// Rules on sizes alone by which a call takes one kernel or another, in plain C++ (a host compiler can check them).
#pragma once

namespace moqe {

// Grouped launches of at most 16 rows: the kernel for few rows (qgemm_few.hip) or a streaming one?  n x k: the experts' matrices; experts_hit: how
// many can have rows, min(S, K); uneven: experts whose weight tiles differ in bytes, or W8A8 ones.
//
// The kernel for few rows starts a work-group per 16 weight rows of an expert, each of which reads its rows' activations again.  That is
// what makes it fast where the launch is a round of work-groups or two, and slow where it is many or the activations outweigh the
// weights: there the streaming kernels' persistent work-groups, which keep them, are the better ones.  us per launch, streaming / few rows (cold weights,
// one expert hit in int4 where nothing else is said):
//   plain, at most 512 work-groups:  4096 x 4096, 16 rows 9.0 / 7.2;  4096 x 11008 22.4 / 15.5;  8192 x 4096, 8 rows 9.4 / 9.3, 16 rows 10.7 / 11.8;
//                                    8192 x 11008, 8 rows 22.9 / 20.1, 16 rows 24.3 / 27.2;  8192 x 2048, 16 rows 8.1 / 7.1
//   plain, up to 2048:               16384 x 512, 4 rows 8.7 / 7.6, 16 rows 8.8 / 11.5;  4096 x 4096, four experts hit, 4 rows 10.8 / 10.6, 16 rows 12.7 / 13.9;
//                                    16384 x 4096, 1 row 13.3 / 13.9, 16 rows 15.3 / 20.3;  32768 x 4096, 1 row 20.5 / 24.3
//   plain, more:                     eight experts hit, 8192 x 4096, 16 rows 39 / 48
//   plain, rows of more than 4096 values: the streaming kernel gives every expert hit the same number of work-groups, so experts of unequal
//                                    bytes keep it waiting: 4096 x 11008, int4, int4, int3 and int8, 4 rows 4.9 us less with few rows, 8 rows 3.5, sixteen experts of
//                                    four formats, 16 rows 11.6 less; of equal bytes 23.8 / 21.1 with 4 rows, 25.7 / 28.7 with 8
//   gate and up (two weight rows to one of activations, and a launch that would else need the bucket kernel ahead of it for k > 4096): a block of
//                                    4096 / 11008, 8 rows 46.7 / 47.1, 16 rows 50.2 / 51.7; of 4096 / 24576, 4 rows 74.4 / 73.7, 16 rows 80.1 / 87.5; four experts hit, 4096 /
//                                    11008, 16 rows 89.3 / 85.5, of equal bytes 4096 / 16384 104.4 / 107.7; eight, 3584 / 18944 237 / 226; sixteen of equal bytes, 4096 /
//                                    11008 171 / 176, 8192 / 8192 270 / 233; 512 / 32768, 16 rows 82.6 / 76.1
constexpr int FEW_MAX_ROWS = 16;
inline bool few_rows_kernel(long long n, long long k, long long rows, int experts_hit, bool gateup, bool uneven) {
  if (rows > FEW_MAX_ROWS) return false;
  if (gateup) {
    const int steps = uneven || k > 4096 ? (experts_hit < 8 ? experts_hit : 8) - 1 : experts_hit > 1;
    return k < 2048 || n * rows < 131072 + 32768 * steps;
  }
  const long long wgs = n / 16 * experts_hit;
  if (wgs <= 512) return n * rows <= 65536 || k <= 2048;
  if (k > 4096) return uneven ? wgs <= 4096 && n * rows <= 131072 : wgs <= 1024 && n * rows <= 16384;
  return wgs <= 2048 && n * rows * k <= (n <= 8192 ? 1ll << 26 : 1ll << 25);
}

// NLP router: whole token rows through the stages between the attentions (router_nlp_rows.hip), or a launch per stage?
//
// Widths: at 512 a work-group holds 32 rows at most, and weights are read too often (9000 rows 279 -> 305 us, 2000 rows of d 16384 339 -> 374,
// where 128 to 384 take 0.45 to 0.85 of the time of a launch per stage).
// Rows: up to 512 the linear kernel shares its k-tiles out over more work-groups than there are tiles of rows (width 384, d 3584, launch per stage /
// whole rows: 100 rows of d 1024 91 / 101 us, 128 rows 102 / 119, 256 107 / 118, 384 111 / 117, 512 122 / 122; 512 of d 16384 132 / 231; narrow ones would
// gain, 256 rows of width 128 86 / 46, width 256 94 / 78).
// Feed-forward: every work-group goes through all of its two matrices, so with the 16 rows apiece that up to 4096 rows are cut into, wide ones are read
// too often (520 to 528 rows of d 1024, launch per stage / whole rows: width 384, feed-forward 6144 182 / 184, 7680 193 / 191, 9216 204 / 215, 12288 245 / 287, 24576 355 / 480;
// width 256, 16384 252 / 245, 24576 334 / 340, 32768 407 / 439; width 128, 16384 242 / 168.  With more rows whole rows gain on it:
// 12288 of width 384, 2304 rows 359 / 365, 4112 rows 365 / 341).
// Input width: every work-group goes through all of W_in too, which pays only while enough of it stays in the caches beside x (launch per stage / whole rows,
// width 384: d 24576, 8192 rows 494 / 412, 32768 rows 1324 / 1153;  d 32768, 4096 rows 537 / 478, 8192 rows 589 / 668, 24576 rows 1320 / 1434;  d 65536, 2048 rows
// 899 / 857, 4096 rows 927 / 1195;  d 131072, 544 rows 1576 / 1421, 1024 rows 1635 / 1778.  Width 256: d 49152, 16384 rows 825 / 730;  d 65536, 8192 rows 922 / 912,
// 12288 rows 959 / 1023.  Width 128: d 65536, 16384 rows 933 / 680).
// The copies' offsets are 32 bits.
inline bool nlp_whole_rows(long long rows, long long d, long long dm, long long d_ff) {
  if (dm > 384 || rows <= 512 || d_ff % dm || dm * (d + 2 * d_ff + 8 * dm) >= (1ll << 30)) return false;
  if (dm == 384 && d > 24576 && rows * d >= (1ll << 27)) return false;
  if (dm == 256 && d > 49152 && rows * d >= (1ll << 29)) return false;
  return rows > 4096 || dm == 128 || d_ff <= (dm == 256 ? 20480 : 7680);
}

}  // namespace moqe
