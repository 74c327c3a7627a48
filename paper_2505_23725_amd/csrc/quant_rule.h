// Which rows the quantised outer update gives a workgroup of their own size (outer.hip).
// Plain arithmetic; it also compiles for the host.
#pragma once

namespace mlc {

// Vectors per thread where a workgroup has just the wavefronts that a row of n elements needs, or 0: a group of 256
// threads takes the row, and may leave most lanes idle in its last vector.
//
// With two vectors a thread a CU holds 16 wavefronts: rows of up to 5120 (5 to a workgroup) and over 6144 (7 and 8)
// nearly fill it, those between (6) three quarters; over 8192 only one workgroup fits, which up to 12288 is
// worse than 256 threads with six vectors.  Beyond, where a thread of 256 would hold eight or twelve vectors,
// it is better by far.  Between 2049 and 8192 the lines
// are where the row-sized workgroup stops being faster, over 1 to 32 replicas, 2 to 8 bits, with and without error
// feedback (ef), each pair of types: its time over that of 256 threads,
//              replicas   1     2     3     4     5     6     8    16    32
//    2056  bf16         1.00  1.00   .93   .91   .90   .93   .92   .93   .89    (256 threads up to two replicas)
//          bf16, ef     1.01  1.00  1.01  1.00  1.02  1.01  1.01  1.03  1.04
//          f32          1.00  1.00  1.04  1.04  1.03  1.04  1.03  1.10  1.10
//    2523  bf16, ragged  1.00  1.00   .95   .95   .94   .95   .96   .94   .91
//    3001  bf16, ragged, ef 1.00 1.00 1.00  1.00  1.00  1.04   .96  1.04  1.06
//    3073  bf16, ragged  1.00 1.01  1.04  1.05  1.06  1.06  1.08  1.10  1.12
//    4104  bf16          .80   .91   .85   .93   .95   .92   .99  1.05  1.07
//    5001  bf16, ragged  .90   .96  1.04  1.06  1.04  1.03  1.05  1.02  1.03
//          f32, ragged   .76   .72   .70   .70   .67   .64   .64   .62   .61    (four vectors a thread spilt there)
//    6152  bf16          .84   .93   .90   .97  1.04  1.01  1.05  1.04   .98
//          bf16, ef      .90   .91   .93   .90   .96   .93   .95   .84   .85
//    8001  bf16, ragged  .79   .82   .88   .90   .91   .94   .95  1.03  1.03
//    8192  bf16          .86   .90   .90   .95  1.01  1.01  1.04  1.09  1.16
//          bf16, ef      .92   .93   .97   .96   .94   .97  1.00  1.02  1.03
//   12296  bf16          .80   .81   .79   .79   .79   .80   .79   .77   .81
//   24576  bf16          .91   .82   .83   .79   .78   .79   .77   .77   .77    (three vectors)
// Ragged rows of four vectors have two wavefronts a SIMD since and no longer spill: of float32 workers, or with a bf16 global copy,
// the row-sized workgroup takes 0.91 to 1.09 of their time now (4201 to 5001 columns, four and eight replicas; 1.29 and 0.83 with
// 16, as few rows fill the last round), and 0.83 to 0.90 with 16 replicas over 6144.
// (The rows of 3073 and of 8192 without feedback are at 8 and 4 bits; rows over 6144 and four replicas take 0.95 of the
// time at 4 bits, 1.00 to 1.03 at 8.)  The mean's second quantisation, another reduction over the row, costs a
// larger workgroup more: 1.03 at each line's last number of replicas without it, 0.98 two below.
// One vector a thread and twice the wavefronts: rows of 2560 to 8192 5 to 45 % slower from four replicas on.
struct QuantRow { long n; int K, bits; bool worker_f32, global_bf16, feedback, second; };

inline int quant_whole_row(const QuantRow& q) {
  if (q.n > 12288) return q.n <= 16384 ? 2 : 3;
  if (q.n <= 2048 || q.n > 8192) return 0;
  int most;                                  // replicas
  if (q.n % 8 != 0) {
    if (q.n <= 4096) return q.n <= 3072 && !q.worker_f32 && q.K >= 3 && q.K <= 5 ? 2 : 0;
    const bool heavy = q.worker_f32 || q.global_bf16;
    most = q.n <= 5120 ? (heavy ? 32 : 2) : q.n <= 6144 ? 2 : heavy ? 32 : 8;
  } else if (q.n <= 4096) {
    if (q.n > 3072 || q.worker_f32 || q.feedback || q.K <= 2) return 0;
    most = 16;
  } else {
    most = q.n <= 5120 ? 6 : q.n <= 6144 ? 2 : q.worker_f32 || q.feedback ? 6 : q.bits < 8 ? 4 : 3;
  }
  return q.K <= (q.second ? most - 2 : most) ? 2 : 0;
}

}  // namespace mlc
