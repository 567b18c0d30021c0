// Which kernel and which block shape a head call takes: plain host arithmetic on sizes, without HIP, so that the launchers
// and the CPU model of the kernels' addresses (tests/test_head_address_model.py) read the same lines.  The kernels themselves and
// what bounds them: head.hip, wide.hip.
#pragma once
#include <stdint.h>

namespace nanospec {

// split-K partial logits of head.hip: at most this many slices of 512 columns, and only while the row count is small, to bound their footprint
constexpr int32_t kSplitMax = 16;
constexpr int32_t kSplitRowsMax = 16384;

// ---- the register-blocked product (wide.hip) ----------------------------------------------------------------------

// its 32-bit byte offsets reach every row
inline bool wide_reaches(int32_t V, int32_t M, int32_t d) { return (int64_t)V * d * 2 <= 0xffffffffll && (int64_t)M * d * 2 <= 0xffffffffll; }

// Which products the register-blocked kernel takes, of those whose rows 32-bit byte offsets reach and that hold_supported and kslice_supported, asked first, leave.  Figures on lists of up to 64 hidden rows are against
// head.hip's kernels.
// More than 16 hidden rows:
//   * any number of rows of one launch's d / 128 steps against two launches of split-K + reduce while that is the shorter walk (d = 1152 6.0 us against 9.6,
//     2048 7.2 against 8.9): d <= 2048, up to 32 hidden rows d <= 1792 (2048: 8.9 against 8.5; from 4096 rows on 0.98);
//   * longer rows from the capacity on at which it beats split-K + reduce, whose workgroups each walk 512 columns only
//     (d = 4096: M = 64, 1000 live rows 11.1 against 9.5 us, 2000: 10.7 / 11.4, 3000: 11.7 / 12.4; M = 24, 2000 live rows
//     11.6 / 10.7, 3000: 12.4 / 13.1);
//   * several sequences, whose split is over their rows together and so finer, from the rows on where the two are even over a quarter, 0.6 and most of the capacity
//     live (this kernel's time over split-K's: d = 4096, 2 of 2560 M = 17 1.19 / 1.05 / 0.82, M = 33 1.13 / 1.02 / 1.16, M = 64 1.04 / 0.94 / 1.10; 8 of 1088 M = 33 1.04 /
//     0.95 / 0.96; d = 8192, 2 of 2560 M = 17 1.45 / 1.15 / 0.86, 8 of 1088 1.27 / 0.85 / 0.94; 8 of 320 M = 33 1.8 / 1.5 / 1.1, 2 of 5120 1.22 / 0.93 / 1.01, M = 64
//     1.11 / 0.90 / 1.14, 8 of 1088 0.92 / 0.95 / 1.02), but for more than 64 hidden rows, which split-K does not take.
// Up to 16 (the kernels of head.hip feed the matrix cores straight from memory, at a quarter of their rate and with the hidden
// rows fetched again for every 16 list rows), where there are rows enough to fill blocks of 32 or 64 with whole hidden-row blocks.  Lists
// are chosen by their capacity; measured with a quarter, half and most of it live (this kernel against head.hip's, whose launches are sized by the capacity
// and so gain most by fewer live rows, except with the K loop of d > 4096, where tiles past the end cost nothing):
//   * one sequence: from the capacity on at which no more is lost with most rows live than is gained with a quarter.  d = 4096, M = 8:
//     capacity 8192 11.3 / 9.2 us with 2000 live rows, 17.0 / 16.5 with 8000; 16384 11.8 / 14.0 and 26.7 / 25.6 (13000); M = 1: 16384 11.3 / 10.0 and
//     26.7 / 23.3, 40960 11.2 / 18.3 and 26.5 / 31.0; M = 16: 9216 11.9 / 13.7 (3000), 24.3 / 22.9 (9000).  d = 2048, M = 8: 8192 7.7 / 5.7 (2000), 16384
//     7.7 / 8.1 and 16.0 / 14.0 (13000).  d = 5120, M = 16: 9216 14.3 / 12.4 (3000), 24576 0.88 to 0.93 of the time from a quarter on;
//   * 8 or more sequences (each die takes one eighth of every list): M = 8 from 65536 rows together (64 sequences of 2300, d = 4096 133 / 147 us, 32 79 / 84, 16
//     of 2300 43 / 46; below, 1.07 to 0.9 of the time); M > 8 from 20480 (8 of 2300, d = 4096 31 / 38; 64 140 / 244);
//   * 2 to 7 sequences: M > 8 only, longer rows than 2048 (d = 4096, 2 of 2000 out of 8192 12.5 / 11.9, of 4000 17.8 / 21.4; M = 12, d = 2048, 4 of
//     4600 out of 9216 1.08 of the time; M = 8, d = 1024, 4 of 2000 7.1 / 6.5, d = 2048 9.8 / 9.2);
//   * 131072 rows together: all but d > 5120 for a few sequences (one list of 147456, d = 4096, M = 1: 30000 live 53 / 87, 100000 160 / 150; d = 8192:
//     3000 live 24.4 / 15.9, 100000 308 / 264);
//   * dense heads where the other kernel's K walk does not fit d -- it works in passes of 1024, 2048 or 4096 columns, zeros included --, and enough rows:
//     M 9 to 16, d no multiple of 2048 (128k rows, M = 16: x 2560 0.74 of the time, x 3584 0.80, x 5120 0.92; M = 9: 0.80, 0.90, 0.99; x 4096 1.08 and so
//     left, but from 13 hidden rows on 0.95; x 2048 0.98 to 1.10, x 6144 1.01 to 1.08; 16400 rows, M = 16 x 3072 0.92, x 1536 1.07, x 5120 0.98);
//     M 5 to 8, d just beyond one pass or two (x 2560 0.94, x 5120 0.91, x 7168 0.95; x 3072, x 3584, x 6144 0.98 to 1.02; below 28000 rows 1.06 to 1.17);
//     d <= 512 (four loads a wavefront would do: 128k rows, M = 1 0.48 against 0.61 of the eight-load form's time, M = 16 0.58 / 0.74; x 768 0.73 / 0.65; x 1024 M = 1
//     0.71 / 0.71, M = 16 0.79 / 0.85).
inline bool wide_supported(int32_t V, int32_t M, int32_t d, int32_t batch, int32_t cap_rows, bool dense) {
  if (!wide_reaches(V, M, d)) return false;
  if (M <= 16) {
    const int64_t rows = (int64_t)cap_rows * batch;
    if (rows > 0x20000000ll) return false;                         // workgroups of one launch
    if (dense) {
      if (d <= 512) return rows >= (M > 8 ? 20480 : 28672);
      if (M <= 4) return false;
      if (d <= 1024) return M > 8 && d > 896 && rows >= 28672;
      if (M <= 8) return rows >= 28672 && ((d > 2048 && d <= 2560) || (d > 4096 && d % 2048 != 0));
      if (d % 2048 != 0) return rows >= (d > 2048 && d < (M > 12 ? 4096 : 3080) ? 16384 : 24576);
      return M > 12 && d == 4096 && rows >= 24576;
    }
    if (rows >= 131072) return d <= 5120 || batch >= 8;
    if (batch >= 8) return M > 8 ? rows >= 20480 : rows >= 65536 && d <= 4096;
    if (batch > 1) return M > 8 && d > 2048 && rows >= 16384;
    if (M > 8) return d <= 5120 && rows >= (d <= 2048 ? 16384 : d <= 4096 ? 9216 : 24576);
    return d <= 4096 && rows >= (M <= 4 ? 24576 : d <= 2048 ? 16384 : 12288);
  }
  const int64_t rows = (int64_t)cap_rows * batch;
  if (rows * ((M + 31) / 32) > 0x40000000ll) return false;         // workgroups of one launch
  if (M > 64 && batch == 1 && rows < 16384) return false;          // many hidden rows on a short list: 64 at a time
  if (d <= (M <= 32 ? 1792 : 2048)) return true;
  if (d <= 2048 || batch == 1 || M > 64 || d > 512 * kSplitMax) return rows >= (M <= 32 ? 4096 : 2560);
  return M <= 32 ? rows >= (d <= 4096 ? 4096 : 8192) : rows * M >= (d <= 4096 ? 262144 : 393216);
}

// Block shapes as (logit rows x hidden rows); kWideGemm is head_gemm_kernel.
enum WideShape : int32_t { kWide32x16, kWide64x16, kWide32x32, kWide64x32, kWide32x64, kWide64x64, kWide128x64, kWide256x128, kWide256x256, kWideGemm, kWideShapes };

// What the shapes are made of: WR x WH wavefronts of FR x FH fragments of 16 x 16 logits, K in steps of BK columns, D register sets.
struct WideBlock {
  int32_t WR, WH, FR, FH, BK, D;
};
constexpr WideBlock kWideBlocks[kWideShapes] = {{2, 1, 1, 1, 128, 4}, {4, 1, 1, 1, 128, 4}, {2, 2, 1, 1, 128, 4}, {4, 1, 1, 2, 128, 2}, {2, 4, 1, 1, 128, 2},
                                                {2, 4, 2, 1, 128, 2}, {4, 1, 2, 4, 64, 2},  {4, 2, 4, 4, 64, 2},  {2, 4, 8, 4, 64, 2},  {2, 4, 8, 4, 64, 2}};

// The block shapes (figures for lists: sequences that share many of their rows).  Up to 64 hidden rows a launch is bound by the bytes a compute unit has in flight over the memory
// latency (few rows) or by HBM (many), so the block grows with the rows: the smallest one while larger blocks would leave
// compute units without work, larger ones to fetch the hidden rows (and, beyond 32 x 32, W_head) less often.  A launch
// only knows the capacity of the lists; thresholds are for live rows around 0.6 of it, dense heads (live == capacity) count double, or less where the
// work is bound by the matrix cores.
//   32 x 32, four register sets of 128 columns: d = 3584, M = 64, 3000 live rows 11.7 us; two sets of 256 columns 12.2;
//     two of 128 13.3; four of 64 13.1; 32 x 64 15.4; 64 x 64 19.8.  With d = 3712 12.3 (split-K + reduce with bounds tests 16.4).
//   32 x 64, eight wavefronts: 4 sequences of 2000 rows, M = 60, d = 4096: 18.1 us; 32 x 32 23.7, 64 x 64 22.6 (slice-loop
//     kernel of head.hip 28.4); at 2 sequences 16.9 against 14.3 for 32 x 32.
//   64 x 64, eight wavefronts: 8 sequences of 2000 rows 25.1 us; 32 x 64 31.5, 32 x 32 38.1, 128 x 64 37.1 (slice-loop kernel
//     36.4); one list of 12000 rows 26.8 against 34.2 / 39.0.
//   128 x 64, four wavefronts, 60 KB of LDS, two workgroups per compute unit: 64 sequences of 2300 rows, d = 2048: 92 us; 64 x 64
//     98 (slice-loop kernel 119); the dense 128k x 4096 head at 48 hidden rows 225 us (64 x 32 blocks 258).
//   up to 32 hidden rows: 32 x 32 (16 sequences of 1500 rows 32 us, slice-loop kernel 49), on long lists and dense 64 x 32 (64
//     sequences of 2000 rows, M = 17: 127 us, slice-loop kernel 196; dense 128k x 4096, M = 24: 205 us, 128 x 64 219, 32 x 32 228;
//     32000 rows 51 / 60 / 59).
//   up to 16: dense and on long lists 64 x 16, on short ones 32 x 16 of two wavefronts (8 sequences of 2300 rows, M = 16: 31 against
//     34.5 us; 64 sequences, M = 8: 141 against 133).
//   dense heads of 33 to 64 hidden rows: 128 x 64 from the rows on that this kernel takes them from (20480 x 2048, M = 64: 64 x 64 takes 1.06 times as long, 17000 x 8192 1.11,
//     16400 0.95).
//   more than 64, one sequence: compute-bound.  64 x 64 blocks while they are few -- rows times blocks of 64 hidden rows --, where larger ones would leave compute
//     units without work.  Against 256 x 128: up to 65536 by capacity, 49152 dense (d = 4096: M = 70, 32000 of 32768 rows 78 / 82 us, 65000 161 / 124; M = 128, 20000 of
//     24576 67 / 79, 30000 of 49152 90 / 86; dense 24000 x 128 0.86 of the time, 36000 1.14); against head_gemm_kernel: 98304, 81920 (M = 130, 20000 of 24576 74 / 83, 30000 of 49152
//     108 / 93; M = 256, 14000 of 24576, d = 2048 41 / 51, 32000 of 32768 146 / 105; M = 512, 10000 of 16448 123 / 88, 32000 of 32768 286 / 119; dense 20480 x 200 79 / 84,
//     24000 x 256 1.1, 16400 x 512 1.6 of the time).
//   then up to 128: 256 x 128 logits, eight wavefronts of 64 x 64;
//   more: head_gemm_kernel; 256 x 256 logits of this kernel (eight wavefronts of 128 x 64, all 160 KB of LDS for the
//     two stages) where d is no multiple of 64 or an operand is not 16-byte aligned.
inline WideShape wide_shape(int32_t M, int32_t d, int32_t batch, int32_t cap_rows, bool dense, bool aligned) {
  const int64_t rows = (int64_t)cap_rows * batch * (dense ? 2 : 1);
  if (M <= 16) return dense || rows >= 131072 ? kWide64x16 : kWide32x16;
  if (M <= 32) return rows < 65536 && !dense ? kWide32x32 : kWide64x32;
  if (M <= 64 || batch > 1) {
    if (rows < 10240) return kWide32x32;
    if (rows < 18432) return kWide32x64;
    return rows < (dense ? 32768 : 98304) ? kWide64x64 : kWide128x64;
  }
  const int64_t work = (int64_t)cap_rows * ((M + 63) / 64);
  if (M <= 128) return work <= (dense ? 49152 : 65536) ? kWide64x64 : kWide256x128;
  if (work <= (dense ? 81920 : 98304)) return kWide64x64;
  return d % 64 == 0 && aligned ? kWideGemm : kWide256x256;
}

// Sequences hold many of the same rows, and a die's L2 sees a row again only if the sequences that hold it run there at the
// same time: for few hidden rows each die takes one eighth of every list (64 sequences of 2300 rows, M = 8: 135 -> 130.5 us, 32: 79
// -> 73.5, 16: 47 -> 43; 8, M = 16: 31.1 -> 29.4), but not where the hidden rows of all sequences, which every die then needs, are as
// many bytes as the rows (64 sequences, M = 16: 140 -> 145; M = 60 on 8 sequences 25 -> 26).  The kernels of head.hip, which fetch all
// hidden rows of a sequence for every 16 list rows, lose by the same order.
inline bool wide_by_die(int32_t M, int32_t batch, int32_t cap_rows, bool dense) {
  const int64_t rows = (int64_t)cap_rows * batch * (dense ? 2 : 1);
  return batch >= 8 && M <= 16 && (M <= 8 || rows < 131072);
}

// Whether the batch-union head always works from the split -- shared rows once against all hidden rows, the rest per sequence: few hidden rows on most rows.  The per-sequence head's time over the
// split's, sequences that draw from one Zipf distribution, M <= 4: 64 of 6000 out of 7000 x 8192 502 / 451, x 4096 251 / 238, x 2048 124 / 119, x 1024 84 / 78; 64 of 2300 out of 5120 x 8192 213 /
// 202, x 4096 103 / 103, x 1024 32 / 37; 32 of 6000 x 8192 264 / 255; 32 of 5120 x 8192 114 / 125.
inline bool union_split(int32_t M, int32_t d, int32_t batch, int32_t cap_rows) { return M <= 4 && d >= 2048 && (int64_t)cap_rows * batch >= 196608; }

// Elsewhere up to 16 hidden rows it is the lists that say: the per-sequence head's workgroups take the same eighth of every list on one die and so find most shared rows in its L2, which is the faster
// way (512 to 8192 columns, 2 to 64 sequences from one Zipf distribution 0.3 to 0.95 of the split's time; 64 of 2300 x 4096, M = 8: 107 / 122 us, 36 of them for the shared rows and 84 for the rest) but
// where the sequences hold nearly the same rows -- samples of one prompt, one candidate set for all -- and there are many pairs of a sequence and a row.  Split over whole lists with 0.7 / 0.8 / 0.9 / 0.95
// / all rows in common: 130000 to 400000 pairs M <= 4 0.82 / 0.71 / 0.62 / 0.57 / 0.45, M = 8 0.90 / 0.80 / 0.76 / 0.72 / 0.57, M = 16 1.02 / 0.93 / 0.89 / 0.86 / 0.78; 65000 to 130000 0.96 / 0.88 / 0.80 / 0.74 / 0.57, 1.03 /
// 0.96 / 0.90 / 0.85 / 0.65, 1.10 / 1.04 / 1.03 / 1.00 / 0.84; 40000 to 65000 1.09 / 1.00 / 0.93 / 0.90 / 0.76, 1.20 / 1.11 / 1.06 / 1.04 / 0.87, 1.19 / 1.06 / 1.03 / 1.05 / 0.77; fewer 1.2 to 1.7.  So the part of the pairs that
// may be left per sequence grows with their number.  More than 16 hidden rows: 1.3 to 1.5, all rows in common 1.07 to 1.2.
constexpr int32_t kUnionPairs = 40960;
inline bool union_feeds(int32_t batch, int32_t cap_rows) { return (int64_t)cap_rows * batch >= kUnionPairs; }
#if defined(__HIPCC__)
__host__ __device__
#endif
inline bool union_split_pairs(int32_t pairs, int32_t rest) {
  return pairs >= kUnionPairs && (int64_t)rest * 524288 <= (int64_t)pairs * (pairs < 196608 ? pairs : 196608);
}

// One list shared by the hidden rows of several sequences (see launch_head_shared): 64 sequences' hidden rows on 7400 rows 36 us with 64 x 64 blocks, 39 with 128 x 64,
// 70 with 256 x 128 (too few workgroups).
inline WideShape wide_shared_shape(int32_t rows_total) { return rows_total <= 16 ? kWide32x16 : rows_total <= 32 ? kWide32x32 : kWide64x64; }

// ---- the kernels of head.hip, up to 64 hidden rows per sequence and launch ----------------------------------------------

// Up to 16 hidden rows: MT row tiles of four hidden rows, KS loads per row and wavefront; head_quad_kernel with NRG row groups of 4 * RT rows
// or, with a K loop, head_quad_private_kernel with 4 * RT rows per workgroup.
struct QuadPlan {
  int32_t MT, KS, NRG, RT;
  bool loop;
};

// Which kernel (all measured on MI355X):
//  * d fits one K-iteration (d <= 512*KS): the shared-hidden-row kernel.  Rows per workgroup follow the
//    row capacity so that small vocabularies still spread over the chip (16 / 8 / 4 rows); with tens
//    of thousands of rows it still wins (dense 128k head, M = 8: 174 us against 188 us barrier-free and
//    184 us for the vendor GEMM library), and for several sequences 2 row groups of 8 rows do best
//    (64 sequences of 2.3k rows: 189 us against 223 us barrier-free).
//  * d needs a K loop: the barrier-free kernel (with a loop the shared form pays two barriers per
//    iteration: 264 us against 118 us at 32k rows of d = 8192, 11.0 against 9.6 us at 1.3k rows).
inline QuadPlan quad_plan(int32_t M, int32_t d, int32_t batch, int32_t cap_rows, bool dense) {
  const int64_t rows = (int64_t)cap_rows * batch;
  QuadPlan q = {(M + 3) / 4, 8, 1, 1, false};
  // No more loads per row and wavefront than d has columns for (a load past d reads column 0 and is multiplied with zeros; eight
  // against two or four: 3000 rows x 8, d = 1024 4.34 -> 3.32 us, d = 2048 5.01 -> 4.47; 349 rows, d = 512 3.34 -> 2.32; 8 sequences
  // of 1500 rows x 8, d = 1024 9.8 -> 7.5).  9..16 hidden rows: 8 loads when that makes d a single K-iteration (up to 128 KB of
  // LDS for the hidden-row operands), else 4.  Up to four on the rows of a dense head, bound by the bytes in flight: eight in half of the wavefronts
  // instead of four in all (100k rows x 2048 and more 0.96 to 0.97 of the time; 65k 0.98, 50k 1.0; x 1536 1.09).
  if (d <= 1024) q.KS = 2;
  else if ((d <= 2048 && !(dense && M <= 4 && d > 1792 && rows >= 65536)) || (M > 8 && d > 4096)) q.KS = 4;
  if (d > 512 * q.KS) {
    // (tiles past the end leave at once in this kernel, so what counts is the live rows: 4 rows per workgroup while they
    // fit 256 workgroups -- about 0.8 of the capacity in the workloads here; 7.0 us at 1000 live rows, 10.1 us at 1091)
    q.loop = true;
    q.RT = rows <= 5 * 256 ? 1 : (q.MT <= 2 || rows < 8192) ? 2 : 4;
    return q;
  }
  if (batch > 1 && rows >= 8192) {
    q.NRG = q.RT = 2;
    return q;
  }
  // 16 / 8 / 4 rows per workgroup: the coarsest shape that still gives every workgroup of the launch (sized by the
  // capacity) a compute unit of its own.  A workgroup without rows costs as much as one with rows here (its loads
  // are unconditional), so one workgroup more than the chip has compute units puts two on one unit and the launch
  // waits for that unit: measured at d = 4096, M = 8, live rows = 0.8 capacity, 8 rows per workgroup: 4.85 us at
  // capacity 2048 (256 workgroups), 6.30 us at 2304 (288); with the earlier thresholds (1440 / 2880 rows) capacity
  // 1280 took 4.88 us (now 4.00) and 2752 took 7.50 us (now 6.52).
  q.NRG = rows > 8 * 256 ? 4 : rows > 4 * 256 ? 2 : 1;
  return q;
}

// Wide trees: split K across workgroups while the rows alone cannot fill the chip.
inline bool head_split(int32_t M, int32_t d, int32_t batch, int32_t cap_rows, bool dense, int64_t partial_bytes, int64_t ld) {
  const int64_t S = (d + 511) / 512;
  return !dense && S >= 2 && S * batch * M * cap_rows * 4 <= partial_bytes && (int64_t)cap_rows * batch <= kSplitRowsMax && cap_rows % 64 == 0 &&
         ld % 4 == 0;
}

// head_tile64_kernel's FAST: 0 = every load tested, 1 = whole slices, hidden rows clamped, 2 = and every wavefront's sixteen hidden rows exist
inline int32_t tile64_fast(int32_t M, int32_t d) { return d % 512 != 0 ? 0 : (M == 64 ? 2 : 1); }

// ---- the hidden rows in registers (hold.hip), up to 16 of them -----------------------------------------------------------

// NW wavefronts of 1024 columns, 8 * parts workgroups per sequence, segments of at most `seg` rows between two sums over the wavefronts.
struct HoldPlan {
  int32_t NW, parts, seg;
};

// How many of the chip's 256 compute units have work on average until the last of `groups` equal workgroups ends, in 1/64.
inline int32_t hold_fill(int64_t groups) { return (int32_t)(groups * 64 / ((groups + 255) / 256 * 256)); }

// Workgroups: one per compute unit while the list's pieces fit that (one list of 8400 x 8192, M = 16: 256 workgroups 29.7 us, 384 33.5, 512 32.2; 30000 x 4096, M = 8:
// 46.0 / 48.8 / 48.6), two of few wavefronts where sequences share them (16 of 5000 x 2048, M = 8: 256 44 us, 512 38).  Numbers of sequences that do not divide
// them leave compute units idle: the most pieces that fit, if they fill three quarters, else the fewest beyond that fill 51 of 64 (48 of 2300 x 4096, M = 8: 384 workgroups 96 us, 768 84;
// 24: 192 59, 384 56).  Dense heads are long enough for the chip to hand them out again as workgroups end (128k x 8192, M = 16: 256 workgroups 358 us, 1024 348;
// 128k x 4096 187 / 186, 512 185).
inline HoldPlan hold_plan(int32_t d, int32_t batch, bool dense) {
  HoldPlan h = {(d + 1023) / 1024, 32, 256};
  if (dense) h.parts = 16 * h.NW;
  else if (batch > 1) {
    const int32_t cu = h.NW <= 2 ? 512 : 256;
    h.parts = cu / (8 * batch);
    if (h.parts < 1 || 8 * batch * h.parts * 4 < cu * 3) {
      h.parts = h.parts < 1 ? 1 : h.parts;
      while (h.parts < 64 && (8 * batch * h.parts < cu || hold_fill(8ll * batch * h.parts) < 51)) ++h.parts;
    }
  }
  return h;
}

inline int64_t hold_lds(const HoldPlan& h, int32_t M) { return (int64_t)h.NW * ((M + 3) / 4 * 4) * (h.seg + 4) * 4; }

// Which products it takes.  Figures: its time over that of the kernels of head.hip and wide.hip with 0.04 / 0.15 / 0.35 / 0.6 / 0.9 of the capacity live, of a batch 0.05 / 0.3 / 0.6 / 0.9.  It is launched over
// the live rows and so gains by lists that are far from full; it loses on few rows, where the others ask for weights before the row count has arrived, where pieces are a few rows for which all hidden rows are
// fetched, and where d leaves its last wavefront's 1024 columns nearly empty.  The others go by steps of the capacity and of the live rows, so that no line has all of the gain on one side: these are drawn for
// the mean over lists that are most often half full or more, not so that none loses (2400 sizes and fills measured for the one-list lines and the batches' before them, K slices' too: 0.87 / 0.78 on the one side, 0.96 on the other;
// 5764 at random measured afterwards 0.78, 45 of them beyond 1.1: 2 of 5504 x 2688, M = 16, 1100 rows 1.26 the most here, 10048 x 5096, M = 61, 4019 rows 1.34 with K slices).
//  One list (capacity):
//   * d >= 5120, M > 4, and d > 4096, M 5 to 8: beyond 5120 (x 8192, M = 16: 5632 1.10 / 1.11 / 1.07 / 0.88 / 0.81, 3072 1.28 / 1.09 / 1.07 / 1.06 / 0.83, 8400 live of 33303 37.8 -> 29.7 us; M = 8: 5632 1.14 / 1.15 /
//     1.08 / 0.94 / 0.90, 3072 1.29 / 1.12 / 1.12 / 1.04 / 0.90; x 6144, M = 12: 5632 1.13 / 1.11 / 1.13 / 0.94 / 0.91, 3072 1.23 / 1.10 / 1.12 / 1.11 / 0.91; M = 8: 5632 0.97 / 0.99 / 0.98 / 1.01 / 0.89, 4160 1.0);
//     M > 8 with d < 5120 from 8192 up to 32768 (x 4224, M = 16: 7168 1.19 / 1.12 / 1.12 / 0.88 / 0.88, 8448 0.92 / 0.92 / 1.03 / 0.91 / 1.03; x 4352, M = 15: 35712 0.73 / 1.21 / 1.04 / 1.01 / 0.95); M <= 4 loses
//     as much as it gains (x 8192: 16384 0.97 / 1.09 at 0.3 / 0.9);
//   * 2048 < d <= 4096: M > 4 beyond 4096, M 5 to 8 with d > 3072 beyond 5120 (x 4096, M = 8: 5632 0.66 / 0.76 / 0.91 / 0.93 / 0.90, 4608 0.66 / 0.73 / 0.88 / 1.09 / 0.89 and 1.14 at 0.75; x 3072: 4608 0.63 / 0.69 /
//     0.81 / 0.98 / 0.91), M > 12 with d < 3072 up to 9216 (x 2560, M = 16: 8448 0.47 / 0.53 / 0.66 / 0.71 / 0.79, 9216 0.79 / 0.84 / 1.05 / 1.15 / 0.88 and 1.20 at 0.75; M = 12: 9216 0.67 / 0.73 / 0.93 / 1.06 / 0.83), d < 4096 up to
//     12288 (x 3072: 20000 1.10 / 0.95 at 0.3 / 0.9); M <= 4 4097 to 6144 and from 12288 on (x 4096: 5120 0.86 / 0.94, 8192 0.93 / 1.07, 16384 0.78 / 1.04 at 0.3 / 0.9);
//   * d = 2048: from 16384 on, M > 8 32768 (M = 8: 16384 0.87 / 0.94, 9000 0.96 / 1.09; M = 16: 65536 0.98 / 0.90, 20000 1.08 / 0.96 at 0.3 / 0.9).
//  Several sequences (capacities together; a die takes the same eighth of every list and finds rows that sequences share in its L2, see wide_by_die).  Lines for lists that draw from one
//  distribution; on 90 sizes in them (2 to 62 sequences, d 2048 to 7936, Zipf draws, 0.3 / 0.55 / 0.8 live) the other kernels take 1.09 of the time on average, up to 1.84 (49 of 1408 x 6144, M = 7 1.30 / 1.66 /
//  1.84; 21 of 4800 x 4480, M = 6 1.6; 19 of 2944 x 4352, M = 5 1.48; 8 of 3200 x 6400, M = 1 1.27).  Lists without rows in common, and nearly empty ones, would have it narrower:
//   * not where a piece is fewer than 16 rows of the capacity (23 of 448 x 6912, M = 4 0.69 / 0.93 / 0.96, 36 of 448 x 2176 0.65 / 0.80 / 1.10);
//   * d > 4096: from 2560 on for four or more, two or three beyond 4096 (x 8192: 4 of 600 out of 1000, M = 8 0.86, 2 of them 1.03; 16 of 2300 out of 5120 0.73, 64 239 -> 217 us; x 5120: 16 of 2300 out of 5120
//     69.6 -> 44.5); M <= 4 where the workgroups fill the chip (24: 1.03); M > 8 and d < 5120 up to 196608 (x 4608, M = 16: 64 of 2300 out of 5120 1.11, 16 0.90);
//   * 2048 < d <= 4096: beyond 4096 (x 4096, M = 8: 8 of 600 out of 1000 0.80, 16 of 2300 out of 5120 0.80, 32 73 -> 59 us, 64 122 -> 107; M = 16: 32 80 -> 64, 64 133 -> 120; 4 of 1000 1.07; x 3072, M = 16: 16 of 600
//     out of 1100 0.64; x 2560, M = 4: 2 of 2300 out of 5120 1.04);
//   * d = 2048: M <= 8 from 16384 on (16 of 2300 out of 5120 0.81, 2 1.05), M > 8 from 65536 on (0.89, 8 of 5120 1.01).
//  Dense heads: M > 8, d of 4096 or 8192, of which a compute unit takes eight wavefronts (128k x 4096, M = 16 207 -> 186 us, M = 9 188 -> 180; 32000 x 8192 104 -> 93; x 5120 1.05, x 2048, M = 9 1.06).
inline bool hold_batch_supported(int32_t M, int32_t d, int32_t batch, int32_t cap_rows) {
  const HoldPlan h = hold_plan(d, batch, false);
  const int64_t rows = (int64_t)cap_rows * batch;
  if (cap_rows < 8 * h.parts * 16) return false;
  if (d > 4096 && rows <= (batch >= 4 ? 2560 : 4096)) return false;
  if (d > 4096 && M <= 4) return hold_fill(8ll * batch * h.parts) >= 51;
  if (d > 4096) return M <= 8 || d >= 5120 || rows < 196608;
  return d > 2048 ? rows > (batch < 4 && M <= 8 && d < 3072 ? 12288 : 4096) : rows >= (M <= 8 ? 16384 : 65536);
}

inline bool hold_supported(int32_t V, int32_t M, int32_t d, int32_t batch, int32_t cap_rows, bool dense) {
  if (M > 16 || d > 8192 || d < 2048 || !wide_reaches(V, M, d)) return false;
  const int64_t rows = (int64_t)cap_rows * batch;
  if (rows > 0x20000000ll) return false;
  if (dense) return M > 8 && (d == 4096 || d == 8192) && rows >= 16384;
  if (batch > 1) return hold_batch_supported(M, d, batch, cap_rows);
  if (d > 4096) return M > 8 && d < 5120 ? rows >= 8192 && rows < 32768 : M > 4 && rows > 5120;
  if (d == 2048) return rows >= (M <= 8 ? 16384 : 32768);
  if (rows <= (M > 4 && M <= 8 && d > 3072 ? 5120 : 4096)) return false;
  if (M <= 4) return rows <= 6144 || rows >= 12288;
  if (M > 12 && d < 3072 && rows >= 9216) return false;
  return d == 4096 || rows <= 12288;
}

// ---- K sliced over the wavefronts (kslice.hip), 17 to 64 hidden rows -------------------------------------------------------

// 8 * LB hidden rows per workgroup (hid_blocks of them), 8 * parts pieces per list, blocks of at most `rows` list rows.  over_*: 2^32 / x rounded up, 0 for 1: n / x is the high
// word of n times it while n * x is below 2^32 (n <= 262144 rows or workgroups, at most 512 pieces, 32 hidden blocks, batch 16).
struct SlicePlan {
  int32_t LB, parts, hid_blocks, rows;
  uint32_t over_hid, over_batch, over_pieces;
};
inline uint32_t slice_reciprocal(uint32_t x) { return x > 1 ? (uint32_t)(((1ull << 32) + x - 1) / x) : 0u; }

// What a workgroup fetches for n rows, list rows (blocks of a multiple of 8, at most 64) and hidden rows together.  Blocks of fewer than 24 list rows cost as if they were larger, and hidden blocks that
// share a piece fetch its rows each for itself, beyond the first 16 rows at half the gain (M = 64, 3000 x 3584, 24 rows + 32 hidden rows 9.35 us, 40 + 24 10.0, 48 + 16 10.4, 16 + 64 11.2; 1000 x 4096: 16 + 16
// 6.3, 16 + 24 6.5, 8 + 32 6.6, 8 + 64 9.2; M = 40, 3000 x 4096: 24 + 24 9.7, 24 + 32 9.3 to 9.8, 16 + 40 10.6; 4 lists of 1500: 48 + 40 13.2, 48 + 24 15.0; M = 64, 8400 x 8192: 40 + 64 42.7, 2 x (40 + 32) 50.8).
// Two workgroups per compute unit take 0.88 of two in turn, as the second one's fetches fill the first one's gaps.
inline int64_t kslice_cost(int64_t n, int64_t LB, int64_t hb, int64_t parts, int64_t batch) {
  const int64_t rows = (n + 8 * parts - 1) / (8 * parts), segs = rows > 64 ? (rows + 63) / 64 : 1, block = ((rows + segs - 1) / segs + 7) / 8 * 8;
  const int64_t each = segs * (10 * (block + 8 * LB) + (block > 16 ? 6 * (hb - 1) * (block - 16) : 0) + (block < 24 ? 10 * (24 - block) : 0));
  const int64_t turns = (8 * parts * hb * batch + 255) / 256;
  return each * turns * (turns > 1 ? 88 : 100);
}

// The cheapest of 256 and 512 workgroups and all widths; the host knows the capacity only, lists are taken for 0.45 and 0.8 full.
inline SlicePlan kslice_plan(int32_t M, int32_t batch, int32_t cap_rows) {
  const int32_t sizes[6] = {8, 6, 5, 4, 3, 2};
  SlicePlan best = {8, 1, 1, 64, 0, 0, 0};
  int64_t least = INT64_MAX;
  for (int i = 0; i < 6; ++i)
    for (int twice = 1; twice <= 2; ++twice) {
      const int64_t LB = sizes[i], hb = (M + 8 * LB - 1) / (8 * LB);
      const int64_t parts = 256 * twice / (8 * hb * batch) > 1 ? 256 * twice / (8 * hb * batch) : 1;
      const int64_t cost = 3 * kslice_cost((int64_t)cap_rows * 9 / 20, LB, hb, parts, batch) + 2 * kslice_cost((int64_t)cap_rows * 4 / 5, LB, hb, parts, batch);
      if (cost < least) {
        least = cost;
        best.LB = (int32_t)LB;
        best.parts = (int32_t)parts;
        best.hid_blocks = (int32_t)hb;
      }
    }
  const int32_t piece = (cap_rows + 8 * best.parts - 1) / (8 * best.parts);
  best.rows = piece > 48 ? 64 : (piece + 7) / 8 * 8;
  best.over_hid = slice_reciprocal(best.hid_blocks);
  best.over_batch = slice_reciprocal(batch);
  best.over_pieces = slice_reciprocal(8 * best.parts);
  return best;
}

// Which products it takes, operands 16-byte aligned (its fetches go straight into LDS).  Figures: its time over that of split-K or the register-blocked product with 0.04 / 0.2 / 0.45 / 0.75 / 0.95 of the
// capacity live; lines drawn as for hold_supported (2050 sizes and fills: 0.78 on the one side, 0.96 on the other):
//  * one list: d >= 1024 up to the capacity at which those fill the chip with larger blocks.  M <= 24: x 2304, M = 17 24576 0.62 / 0.86 / 0.81 / 0.93 / 1.0, 32768 1.0 / 1.21 / 1.07 / 1.02 / 0.95; x 5120,
//    M = 24 24576 0.57 / 0.93 / 0.81 / 0.88 / 0.95, 32768 0.98 / 1.29 / 1.03 / 0.99 / 0.93.  M 25 to 32: x 3584, M = 32 32768 0.65 / 0.98 / 0.92 / 1.0 / 0.93, 40960 1.05 / 1.36 / 0.93 / 0.98 / 1.01.  M <= 32, x 2048: M = 17 20480
//    0.69 / 0.85 / 0.82 / 1.07 / 1.07, 24576 0.69 / 0.92 / 0.94 / 1.05 / 1.13.  M > 32: x 4096, M = 64 20480 0.49 / 0.70 / 0.91 / 1.07 / 0.91, 40960 1.0 on average; x 2048, M = 64 20480 0.65 / 0.75 / 0.96 / 1.10 / 1.03; x 1024, M = 48
//    16384 0.80 / 0.83 / 1.04 / 0.93 / 1.0, 20480 0.62 / 0.70 / 0.97 / 1.12 / 1.06, M = 64 5120 0.88, 10240 0.86 / 0.81 / 1.01 / 1.13 / 0.93.  x 512: up to 2600 M = 32 0.81 to 0.87, M = 64 0.84 to 0.96, 8200 1.04;
//  * but few long rows, which split-K spreads over more of the chip (x 8192, M = 17 640 1.17 / 1.14 / 1.09 / 1.04 / 1.0, 1280 1.17 / 1.13 / 0.93 / 0.86 / 0.85; M = 64 640 1.08 / 1.04 / 0.98 / 0.91 / 0.88, 1280 0.99 / 1.0 / 0.84 /
//    0.79 / 0.87; x 7168, M = 17 640 1.07 / 1.07 / 1.04 / 0.99 / 0.95, 1280 1.08 / 1.08 / 0.88 / 0.80 / 0.80; x 6144 0.91 to 0.99);
//  * several: while 205 of 256 workgroups can be had for equal shares and the work is little (4 of 600 out of 1000 x 4096 0.63 to 0.69, of 2300 out of 5120 0.68 to 0.87; 8 of 3500, M = 20 0.83, M = 64 1.06; 12 of
//    600 1.0 to 1.1; 16 of 1280 M = 48 0.73 to 0.89; 24 of 600 1.1 to 1.7), 28672 rows together (2 of 20480 x 4096, M = 17 1.26 with 0.2 live), d <= 2048 and M > 32 20480 (2 of 14336 x 2048, M = 33 1.16 with 0.95); not where pieces are
//    few rows beside many hidden rows -- more than twelve sequences with M > 48 below 1024 rows each (16 of 640 x 3584, M = 64 0.97 / 1.01 / 1.12 / 1.12 / 0.75, of 256 1.13 to 1.30), below 400 d > 6144 (8 of 320 x 8192, M = 48 1.27 / 1.26 /
//    1.14 / 0.87 / 0.83; 14 1.65 / 1.51 / 1.06 / 0.95 / 0.82) and d >= 3072 with more than eight and M > 32 (16 of 320 x 5120, M = 48 1.29 / 1.19 / 1.01 / 0.79 / 0.75);
//  * no dense heads (128k x 4096 1.01 to 1.15, 32000 x 4096 1.0 to 1.1, x 8192 0.92 to 0.99, 128k x 8192 1.02 to 1.2, x 1024 1.2 to 1.3).
inline bool kslice_supported(int32_t V, int32_t M, int32_t d, int32_t batch, int32_t cap_rows, bool dense, bool aligned) {
  if (M <= 16 || M > 64 || d < 512 || dense || !aligned || !wide_reaches(V, M, d)) return false;
  const int64_t rows = (int64_t)cap_rows * batch;
  if (d < 1024) return rows <= 3072;
  if (batch > 1) {
    if (batch > 16 || 256 / (8 * batch) * (8 * batch) < 205) return false;
    if (cap_rows < 1024 && batch > 12 && M > 48) return false;
    if (cap_rows < 400 && (d > 6144 || (d >= 3072 && batch > 8 && M > 32))) return false;
    return rows <= (d <= 2048 && M > 32 ? 20480 : 28672) && rows * M <= (d < 2048 ? 700000 : batch <= 8 ? 1400000 : 1000000);
  }
  if (rows < 1024 && (d > 7168 || (d > 6144 && M <= 32))) return false;
  if (M <= 32) return rows <= (d <= 2048 ? 20480 : M <= 24 ? 24576 : 32768);
  return rows <= (d >= 2048 ? 20480 : M <= 48 ? 16384 : 8192);
}

// ---- stream initialisation (vocab.hip) -------------------------------------------------------------------------------------

constexpr int32_t kInitFewSeqs = 16;           // more fill the chip with larger id ranges

// One launch of one workgroup per sequence (vocab_init_kernel) or the id ranges counted all over the chip (two launches, three for long prompts).
// The former's time grows with the prompt -- the additions to the counters, a frequent token's all to one address in L2, about 0.7 us per 100 tokens -- and with the
// stream it replaces, whose ring of up to `window` tokens it undoes one scattered store each, 0.26 us per 1024; the host knows the window only.  The latter's is as good as
// constant, and grows with the sequences.  V = 128256, |T| = 2000, initialisations back to back over a stream that filled the window, one launch / ranges, us: one
// sequence, window 1024, 64 tokens 5.8 / 6.9, 600 9.8 / 7.6; window 8192, 64 tokens 7.9 / 7.3; 16384 10.2 / 6.9; 65536 25 / 7.2; 235312 75 / 7.4; 64 sequences, window 1024, 1024 tokens 13.9 /
// 18.4; 8192, 600 15.9 / 17.2, 1500 21.7 / 18.8; 65536, 64 37 / 15; 235312 125 / 15.  In front of a draft step the second launch costs about 3 us more than that (requests of
// one sequence and 192 to 331 tokens 1.8 to 3.4 us, of three and 214 to 463 2.5 to 3.2), so the lines for a small window are 640 and 1536 tokens.
inline bool vocab_init_serial(int32_t batch, int32_t window, int32_t longest) { return longest + window / 24 <= (batch <= kInitFewSeqs ? 640 : 1536); }

// ---- selection from rows that one workgroup's registers do not hold (topk.hip) --------------------------------------------------

constexpr int32_t kTopkChunk = 16384;          // elements per workgroup in the two-pass top-k

// How many ids a list is likely to hold, of which the launcher knows only the capacity: a candidate set is as large as the room made for it, a queue of distinct
// ids fills its window, and a window of raw tokens holds about a sixth of its length (Zipf streams: 8400 of 33k, 32800 of 235k).
inline int64_t topk_expected(int32_t topk_cap, int32_t window, bool distinct) { return (int64_t)topk_cap + (distinct ? window : window / 6); }

// Chunks of every row all over the chip and a second launch that merges their winners, or one workgroup per row (which walks it, or, a list of up to 16384 live
// ids, selects it at once; in chunks such a list waits for the second launch).  Measured, one workgroup / chunks, us: 8 rows, k = 10, 3000 ids 5.1 / 6.3, 17000 10.3 /
// 8.4, 50000 14.7 / 9.9, 128000 22.2 / 9.1; k = 1, 32000 10.5 / 8.1; k = 16, 128000 23.3 / 9.4; 64 rows, k = 10, 32000 11.1 / 10.1, 128000 22.2 / 16.8; 88 rows 128000 23.3 /
// 22.5, 64 dense rows 23 / 19, 128 21 / 28, 1024, k = 3 97 (5.4 TB/s; rows of 128255 the same) / 202 (381).  Larger k: 8 rows, k = 40, 32000 12.4 / 10.9, 17000 13.0 / 41 (a last
// chunk of fewer than 16 k elements goes the slow way), 80000 21.7 / 14.5, 128000 34.8 / 21.2.
inline bool topk_chunks(bool list, int64_t rows, int32_t k, int64_t expected) {
  if (!list) return rows < 96;
  return rows <= 64 && expected > (k <= 16 ? kTopkChunk : 65536);
}

}  // namespace nanospec
