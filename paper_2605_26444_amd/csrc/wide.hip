// Eq. 1 of the paper (Sec. 3.1) for many hidden rows at once -- the dense comparison point of a wide draft tree
// (64 hidden rows) and of a batch of sequences (hundreds) -- as a register-blocked matrix-core product.
//
// The kernels of head.hip give every wavefront one 16-row tile of W_head and stream all hidden rows past it: each
// matrix instruction then needs 1.25 KB of operands out of LDS, 2.5 times what LDS delivers at the matrix cores'
// rate, and W_head is read once per 64 hidden rows.  Here a workgroup owns a BM x BN block of the logits (BM rows
// of W_head, BN hidden rows) and walks K in steps of BK columns: both operand blocks of a step are fetched with
// 16-byte loads into registers two steps ahead, parked in padded LDS (two stages, one barrier per step), and every
// wavefront multiplies an (FR*16) x (FH*16) sub-block, so one operand fragment read from LDS feeds FH (or FR)
// matrix instructions.  W_head is read once per BN hidden rows.
#include "common.h"

namespace nanospec {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_u __attribute__((aligned(4)));   // global memory takes 16-byte stores at any 4-byte address

constexpr int kWidePad = 32;     // bytes between LDS rows: rows r and r+4 share banks, the 16 lanes of a fragment read never meet

// WR x WH wavefronts (4 or 8); a wavefront owns FR x FH fragments of 16 x 16 logits.
//   logits[m][j] for hidden row m < M and list row j < n, row stride ld.  ids == nullptr: rows 0..n-1.
//   opos != nullptr ([opos_len], a multiple of 4 entries): row j's logits go to column opos[j] instead, nowhere if negative.
//   seq_rows > 0: one list for the hidden rows of several sequences, seq_rows each, with columns of their own ([..][ids_stride]).
// d % BK == 0 (checked by the launcher).  Rows past n read row 0, hidden rows past M read row M-1; neither is stored.
// Workgroup order: the chip hands consecutive workgroups to its eight dies in turn and each die has its own L2, so
// the hidden-row blocks of one row block run back to back on one die (blk -> (row block, hidden block) below)
// and find the row block's weights in that L2.
// Several sequences (batch > 1): list, row count, hidden rows, logits and columns of sequence b lie at b times their
// strides, and the sequences take turns (sequence fastest), so that one die works for few sequences and keeps their
// hidden rows in its L2.
// TAIL: any d % 8 == 0 -- the last step's pieces past column d are fetched from column 0 and parked as zeros, and the
// number of steps may be odd.  Without it d % (D * BK) == 0.
template <int WR, int WH, int FR, int FH, int BK, int D, bool TAIL>
__device__ __forceinline__ void wide_block(const uint32_t blk, const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, const int32_t* __restrict__ ids,
                                           const int32_t* __restrict__ n_dev, int n_fixed, int V, int batch, int M, int d, int64_t ld, int64_t ids_stride,
                                           float* __restrict__ logits, int row_blocks, int hid_blocks, const int32_t* __restrict__ opos, int opos_len,
                                           int seq_rows, int by_die) {
  constexpr int NT = 64 * WR * WH;
  constexpr int BM = WR * FR * 16, BN = WH * FH * 16;
  constexpr int CPR = BK / 8;                      // 16-byte pieces per row and step
  constexpr int RPP = NT / CPR;                    // rows one pass of the workgroup's threads covers
  constexpr int NA = BM / RPP, NB = BN / RPP;      // passes over the W block / the hidden-row block
  constexpr int STR = BK * 2 + kWidePad;           // LDS row stride in bytes
  constexpr int STAGE = (BM + BN) * STR;
  static_assert(BM % RPP == 0 && BN % RPP == 0, "whole passes");
  static_assert(D >= 2 && D % 2 == 0, "step s reads LDS stage s & 1: the unrolled group of D steps must keep that parity");
  extern __shared__ __attribute__((aligned(16))) char smem[];

  // blk -> die x = blk % 8, slot r = blk / 8; hidden block = r % hid_blocks, row block = (r / hid_blocks) * 8 + x
  // several sequences: sequence = blk % batch, hidden block and row block follow; by_die: die x takes the x-th eighth of every
  // sequence's row blocks (the cuts move by up to a block from sequence to sequence, so that the eighths even out)
  int b = 0, hb, rb, n;
  if (batch == 1) {
    const int xq = blk & 7, xr = blk >> 3;
    hb = xr % hid_blocks;
    rb = (xr / hid_blocks) * 8 + xq;
    n = n_dev ? n_dev[0] : n_fixed;
  } else {
    const int x = blk & 7, xr = by_die ? blk >> 3 : blk;
    hb = by_die ? xr % hid_blocks : xr / batch % hid_blocks;
    b = (by_die ? xr / hid_blocks : xr) % batch;
    rb = xr / batch / hid_blocks;
    n = n_dev ? n_dev[b] : n_fixed;
    if (by_die) {
      const int blocks = (n + BM - 1) / BM, end = ((x + 1) * blocks + (b & 7)) >> 3;
      rb += (x * blocks + (b & 7)) >> 3;
      if (rb >= end) return;
    }
  }
  if (rb >= row_blocks) return;
  const int j0 = rb * BM, m0 = hb * BN;
  if (j0 >= n) return;

  if (ids) ids += b * ids_stride;
  if (opos) opos += b * ids_stride;
  H += (int64_t)b * M * d;
  logits += (int64_t)b * M * ld;

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wr = w / WH, wh = w % WH;
  const int pc = tid % CPR, pr = tid / CPR;        // this thread's 16-byte piece and first row of a pass

  // byte offsets of this thread's rows from W and H (below 4 GB each: checked by the launcher)
  uint32_t aoff[NA], boff[NB];
  int rowv[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int j = j0 + pr + i * RPP;
    rowv[i] = j < n ? j : j0;                      // a row past the end is a copy of the block's first row, never stored
  }
  if (ids) {                                        // one uniform branch around all of them: the loads go out together
#pragma unroll
    for (int i = 0; i < NA; ++i) rowv[i] = ids[rowv[i]];
  }
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    int64_t row = rowv[i];
    row = row < 0 ? 0 : (row >= V ? V - 1 : row);
    aoff[i] = (uint32_t)(row * d * 2);
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    int m = m0 + pr + i * RPP;
    m = m < M ? m : M - 1;
    boff[i] = (uint32_t)((int64_t)m * d * 2);
  }
  const char* Wb = reinterpret_cast<const char*>(W);
  const char* Hbase = reinterpret_cast<const char*>(H);

  // D register sets: the loads of step s+D are issued before the matrix work of step s starts, so a load has D
  // steps' time to arrive (one step of matrix work is shorter than an HBM round trip) and D-1 sets -- (D-1) x (BM+BN)
  // x BK x 2 bytes -- are in flight per workgroup all the time
  u32x4 ga[D][NA], gb[D][NB];
  auto fetch = [&](int ks, int set) {
    uint32_t off = (uint32_t)ks * BK * 2 + pc * 16;
    if (TAIL && off >= (uint32_t)d * 2) off = 0;    // past the end of the row: its start instead, parked as zeros
#pragma unroll
    for (int i = 0; i < NA; ++i) ga[set][i] = *reinterpret_cast<const u32x4*>(Wb + (aoff[i] + off));
#pragma unroll
    for (int i = 0; i < NB; ++i) gb[set][i] = *reinterpret_cast<const u32x4*>(Hbase + (boff[i] + off));
  };
  auto park = [&](int stage, int set, int ks) {
    char* As = smem + stage * STAGE;
    char* Bs = As + BM * STR;
    if (TAIL && ks * BK + BK > d) {                 // uniform: only the last step
      const bool in = ks * BK + pc * 8 < d;
      const u32x4 zero = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int i = 0; i < NA; ++i) ga[set][i] = in ? ga[set][i] : zero;
#pragma unroll
      for (int i = 0; i < NB; ++i) gb[set][i] = in ? gb[set][i] : zero;
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) *reinterpret_cast<u32x4*>(As + (pr + i * RPP) * STR + pc * 16) = ga[set][i];
#pragma unroll
    for (int i = 0; i < NB; ++i) *reinterpret_cast<u32x4*>(Bs + (pr + i * RPP) * STR + pc * 16) = gb[set][i];
  };

  f32x4 acc[FR][FH];
#pragma unroll
  for (int a = 0; a < FR; ++a)
#pragma unroll
    for (int b = 0; b < FH; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  // fragment addresses: lane = row (mod 16) + 16 * k group, 8 consecutive k (16 bytes) per lane
  const int frag_off = (lane & 15) * STR + (lane >> 4) * 16;
  // One step: BK/32 sub-steps of FR x FH matrix instructions.  Operand fragments are asked for one fragment ahead
  // of their use (the next row fragment while the current one's FH instructions run, the next sub-step's hidden-row
  // fragments during the last row fragment), so an LDS round trip is covered by matrix work of the same wavefront.
  auto multiply = [&](int stage) {
    const char* As = smem + stage * STAGE + (wr * FR * 16) * STR + frag_off;
    const char* Bs = smem + stage * STAGE + BM * STR + (wh * FH * 16) * STR + frag_off;
    constexpr int KK = BK / 32;
    if constexpr (WR * WH != 8) {                     // four wavefronts, memory-bound: the plain order, scheduled by the compiler (205 against 217 us)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        bf16x8 bq[FH];
#pragma unroll
        for (int b = 0; b < FH; ++b) bq[b] = *reinterpret_cast<const bf16x8*>(Bs + b * 16 * STR + kk * 64);
#pragma unroll
        for (int a = 0; a < FR; ++a) {
          const bf16x8 aq = *reinterpret_cast<const bf16x8*>(As + a * 16 * STR + kk * 64);
#pragma unroll
          for (int b = 0; b < FH; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, bq[b], acc[a][b], 0, 0, 0);
        }
      }
      return;
    }
    bf16x8 bf[2][FH], af[2];
#pragma unroll
    for (int b = 0; b < FH; ++b) bf[0][b] = *reinterpret_cast<const bf16x8*>(Bs + b * 16 * STR);
    af[0] = *reinterpret_cast<const bf16x8*>(As);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
      for (int a = 0; a < FR; ++a) {
        const int cur = (kk * FR + a) & 1;
        if (a + 1 < FR) {
          af[cur ^ 1] = *reinterpret_cast<const bf16x8*>(As + (a + 1) * 16 * STR + kk * 64);
        } else if (kk + 1 < KK) {
          af[cur ^ 1] = *reinterpret_cast<const bf16x8*>(As + (kk + 1) * 64);
#pragma unroll
          for (int b = 0; b < FH; ++b) bf[(kk + 1) & 1][b] = *reinterpret_cast<const bf16x8*>(Bs + b * 16 * STR + (kk + 1) * 64);
        }
#pragma unroll
        for (int b = 0; b < FH; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[cur], bf[kk & 1][b], acc[a][b], 0, 0, 0);
      }
    }
    // The order above is the order wanted; left alone, the scheduler puts every fragment read right in front of its
    // first use.  Groups: the LDS reads of the next fragment(s), then FH matrix instructions.  For the shapes of eight
    // wavefronts, of which the compute-bound ones gain: 644 -> 614 us at 512 hidden rows on 256 x 128 logits.  The 32 x 64 and
    // 64 x 64 shapes are memory-bound and do not care (16 sequences of 64 x 2000 rows, d = 3584: 46.8 with, 46.7 without);
    // the four-wavefront shapes lose with it (205 -> 218 us at 64 hidden rows).
    if constexpr (WR * WH == 8) {
      __builtin_amdgcn_sched_group_barrier(0x100, FH + 1, 0);
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
        for (int a = 0; a < FR; ++a) {
          if (a + 1 < FR) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          else if (kk + 1 < KK) __builtin_amdgcn_sched_group_barrier(0x100, FH + 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, FH, 0);
        }
      }
    }
  };

  // Every fetch is unconditional -- past the end the last step is fetched again and never used -- because a load
  // under a branch makes the number of loads in flight unknowable at compile time, and every wait for one register
  // set then becomes a wait for all of them.  Set s % D receives step s + D right after it was parked for step s.
  // Without TAIL and with D == 2, nk is even and the loop body has no branch at all; else any nk, and the steps past the
  // end skip their matrix work (a uniform branch around LDS reads and matrix instructions only).
  const int nk = (d + BK - 1) / BK;
#pragma unroll
  for (int j = 0; j < D; ++j) fetch(j < nk ? j : nk - 1, j);
  __builtin_amdgcn_sched_barrier(0);
  park(0, 0, 0);
  __syncthreads();
  for (int ks = 0; ks < nk; ks += D) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const int st = ks + j;                        // LDS stage j & 1 holds this step, set (j + 1) % D holds (or awaits) the next
      fetch(st + D < nk ? st + D : nk - 1, j);
      __builtin_amdgcn_sched_barrier(0);            // the loads go out before the matrix work, not after it
      if ((D == 2 && !TAIL) || st < nk) multiply(j & 1);
      park((j + 1) & 1, (j + 1) % D, st + 1 < nk ? st + 1 : nk - 1);               // that stage's last readers passed the previous barrier
      __syncthreads();
    }
  }

  // result lane l holds list rows j + v (v = 0..3), j = 4 * (l / 16), of hidden row l % 16 of the fragment
#pragma unroll
  for (int a = 0; a < FR; ++a) {
    const int j = j0 + (wr * FR + a) * 16 + 4 * (lane >> 4);
#pragma unroll
    for (int b = 0; b < FH; ++b) {
      const int m = m0 + (wh * FH + b) * 16 + (lane & 15);
      if (m >= M || j >= n) continue;
      float* dst = logits + (int64_t)m * ld + j;
      if (opos) {                                       // rows kept in an order of their own: list row j's logits go to column opos[j]
        const int32_t* col = opos + (seq_rows ? (int64_t)(m / seq_rows) * ids_stride : 0);
        const int4 jo4 = j + 3 < opos_len ? *reinterpret_cast<const int4*>(col + j) : make_int4(-1, -1, -1, -1);
        const int jo[4] = {jo4.x, jo4.y, jo4.z, jo4.w};
        float* rowp = logits + (int64_t)m * ld;
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (j + v < n && jo[v] >= 0) rowp[jo[v]] = acc[a][b][v];
      } else if (j + 3 < n) {
        *reinterpret_cast<f32x4_u*>(dst) = acc[a][b];
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (j + v < n) dst[v] = acc[a][b][v];
      }
    }
  }
}

template <int WR, int WH, int FR, int FH, int BK, int D, bool TAIL>
__global__ __launch_bounds__(64 * WR * WH) void head_wide_kernel(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H,
                                                        const int32_t* __restrict__ ids, const int32_t* __restrict__ n_dev, int n_fixed,
                                                        int V, int batch, int M, int d, int64_t ld, int64_t ids_stride,
                                                        float* __restrict__ logits, int row_blocks, int hid_blocks,
                                                        const int32_t* __restrict__ opos, int opos_len, int seq_rows, int by_die) {
  wide_block<WR, WH, FR, FH, BK, D, TAIL>(blockIdx.x, W, H, ids, n_dev, n_fixed, V, batch, M, d, ld, ids_stride, logits, row_blocks, hid_blocks, opos, opos_len, seq_rows, by_die);
}

// The list that several sequences share.  Often it is empty -- the device says whether it is used at all --, so its launch is no more workgroups than the chip holds, each of
// which takes every gridDim.x-th block (a multiple of 8 blocks apart: on one die) up to the list's end.  The last barrier of a block's K walk stands between its LDS and the next block's.
// An empty list of 5120 places in front of 64 sequences of 2300 x 4096, M = 8: 2.25 us with 512 workgroups, 2.8 with one for each block that there is room for.
template <int WR, int WH, int FR, int FH, int BK, int D, bool TAIL>
__global__ __launch_bounds__(64 * WR * WH) void head_wide_shared_kernel(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, const int32_t* __restrict__ ids,
                                                                        const int32_t* __restrict__ n_dev, int V, int M, int d, int64_t ld, int64_t opos_stride,
                                                                        float* __restrict__ logits, int row_blocks, int hid_blocks,
                                                                        const int32_t* __restrict__ opos, int opos_len, int seq_rows) {
  const int n = n_dev[0], used = (n + WR * FR * 16 - 1) / (WR * FR * 16);
  const uint32_t blocks = (uint32_t)((used < row_blocks ? used : row_blocks) + 7) / 8 * 8 * hid_blocks;
  for (uint32_t blk = blockIdx.x; blk < blocks; blk += gridDim.x)
    wide_block<WR, WH, FR, FH, BK, D, TAIL>(blk, W, H, ids, nullptr, n, V, 1, M, d, ld, opos_stride, logits, row_blocks, hid_blocks, opos, opos_len, seq_rows, 0);
}

template <int WR, int WH, int FR, int FH, int BK, int D>
static hipError_t run_wide_shared(const uint16_t* W, const uint16_t* H, const int32_t* ids, const int32_t* n_dev, int32_t cap_rows, int32_t V, int32_t M, int32_t d, int64_t ld,
                                  int64_t opos_stride, float* logits, const int32_t* opos, int32_t seq_rows, hipStream_t s) {
  constexpr int BM = WR * FR * 16, BN = WH * FH * 16;
  constexpr int LDS = 2 * (BM + BN) * (BK * 2 + kWidePad), kResident = 256 * (160 * 1024 / LDS < 4 ? 160 * 1024 / LDS : 4);
  const int row_blocks = (cap_rows + BM - 1) / BM, hid_blocks = (M + BN - 1) / BN;
  const int64_t blocks = (int64_t)((row_blocks + 7) / 8) * hid_blocks * 8;
  if (blocks > 0x7fffffff - kResident || !wide_reaches(V, M, d)) return hipErrorInvalidValue;
  const unsigned grid = blocks < kResident ? (unsigned)blocks : kResident;
  if (d % (D * BK) == 0)
    head_wide_shared_kernel<WR, WH, FR, FH, BK, D, false><<<dim3(grid), 64 * WR * WH, LDS, s>>>(W, H, ids, n_dev, V, M, d, ld, opos_stride, logits, row_blocks, hid_blocks, opos,
                                                                                              cap_rows / 4 * 4, seq_rows);
  else
    head_wide_shared_kernel<WR, WH, FR, FH, BK, D, true><<<dim3(grid), 64 * WR * WH, LDS, s>>>(W, H, ids, n_dev, V, M, d, ld, opos_stride, logits, row_blocks, hid_blocks, opos,
                                                                                             cap_rows / 4 * 4, seq_rows);
  return hipGetLastError();
}

template <int WR, int WH, int FR, int FH, int BK, int D>
static hipError_t run_wide(const uint16_t* W, const uint16_t* H, const int32_t* ids, const int32_t* n_dev, int32_t n_fixed, int32_t cap_rows,
                           int32_t V, int32_t batch, int32_t M, int32_t d, int64_t ld, int64_t ids_stride, float* logits, const int32_t* opos,
                           int32_t seq_rows, int by_die, hipStream_t s) {
  constexpr int BM = WR * FR * 16, BN = WH * FH * 16;
  constexpr int LDS = 2 * (BM + BN) * (BK * 2 + kWidePad);
  const int row_blocks = (cap_rows + BM - 1) / BM, hid_blocks = (M + BN - 1) / BN;
  const int64_t grid = batch == 1 ? (int64_t)((row_blocks + 7) / 8) * hid_blocks * 8
                       : by_die     ? (int64_t)((row_blocks + 7) / 8) * hid_blocks * batch * 8
                                    : (int64_t)row_blocks * hid_blocks * batch;
  if (grid > 0x7fffffff || (int64_t)V * d * 2 > 0xffffffffll || (int64_t)M * d * 2 > 0xffffffffll) return hipErrorInvalidValue;
  if (d % (D * BK) == 0)
    head_wide_kernel<WR, WH, FR, FH, BK, D, false><<<dim3((unsigned)grid), 64 * WR * WH, LDS, s>>>(
        W, H, ids, n_dev, n_fixed, V, batch, M, d, ld, ids_stride, logits, row_blocks, hid_blocks, opos, cap_rows / 4 * 4, seq_rows, by_die);
  else
    head_wide_kernel<WR, WH, FR, FH, BK, D, true><<<dim3((unsigned)grid), 64 * WR * WH, LDS, s>>>(
        W, H, ids, n_dev, n_fixed, V, batch, M, d, ld, ids_stride, logits, row_blocks, hid_blocks, opos, cap_rows / 4 * 4, seq_rows, by_die);
  return hipGetLastError();
}

constexpr int kGemmStage = 4 * 128 * 128;        // bytes of one stage: A0, A1, B0, B1 (128 rows x 128 bytes each)

// operands by lds_fetch16 (global_load_lds, common.h) and counted waits
#define NS_WAIT_VM(n) asm volatile("s_waitcnt vmcnt(" #n ")" ::: "memory")
#define NS_BARRIER()                        \
  do {                                      \
    __builtin_amdgcn_sched_barrier(0);      \
    asm volatile("" ::: "memory");          \
    __builtin_amdgcn_s_barrier();           \
    asm volatile("" ::: "memory");          \
    __builtin_amdgcn_sched_barrier(0);      \
  } while (0)

// The compute-bound product: more than 128 hidden rows of one sequence on many rows, d a multiple of 64.
// 256 x 256 logits per workgroup of eight wavefronts (128 x 64 each), K in 64-column steps, two LDS stages of 64 KB.  What it has
// to do per step on a compute unit is 2048 cycles of matrix work (of one SIMD) and as many cycles of LDS (192 KB of
// fragment reads, 64 KB of fills), so everything has to overlap:
//   * the operand blocks go from memory straight into LDS (no registers, no LDS write instructions), 14 to 16 KB pieces at a
//     time, one step and a quarter to one and three quarters ahead of their use.  The 16-byte pieces of a row are stored
//     permuted by the row's low three bits (the fetching lanes permute their addresses), so that neither side has bank
//     conflicts without padding;
//   * a step is four phases, each a quarter of the block (row half x hidden half) of 16 matrix instructions per wavefront, and the
//     second four wavefronts run one phase half behind the first: while one wavefront of a SIMD multiplies, the other one
//     asks for its next fragments (the eight-wavefront ping-pong schedule published for this chip, HipKittens, arXiv 2511.08083;
//     the split of the fetches, the permutation, the phases and the waits are this kernel's).  Fragments are asked for one barrier
//     before they are needed;
//   * a piece of LDS is refilled one phase after all its readers have consumed it (the barriers between say so), and is read
//     after every wavefront has waited for its own fetches of it (the counted waits, then a barrier).
// 1024 hidden rows on the 128k x 4096 matrix: 896 us = 1.20 PFLOP/s (head_wide_kernel's 256 x 256 shape: 1036); the loop takes
// 1.16 times its matrix cycles, at the 1.7 GHz this load runs at.  512 hidden rows 532 -> 490 us, 130: 309 -> 275.  The
// sums are taken in the same order: results are bit-equal.
__global__ __launch_bounds__(512, 2) void head_gemm_kernel(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H,
                                                           const int32_t* __restrict__ ids, const int32_t* __restrict__ n_dev, int n_fixed,
                                                           int V, int M, int d, int64_t ld, float* __restrict__ logits, int row_blocks,
                                                           int hid_blocks, const int32_t* __restrict__ opos, int opos_len) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int xq = blockIdx.x & 7, xr = blockIdx.x >> 3;
  const int hb = xr % hid_blocks, rb = (xr / hid_blocks) * 8 + xq;
  if (rb >= row_blocks) return;
  const int n = n_dev ? n_dev[0] : n_fixed;
  const int j0 = rb * 256, m0 = hb * 256;
  if (j0 >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = w >> 2, wh = w & 3;

  // this lane's pieces: instruction i of half h covers rows (2w + i) * 8 + lane / 8 of the half
  const int pc = (lane & 7) ^ (lane >> 3);                 // row & 7 == lane >> 3 in every instruction: the swizzled piece
  uint32_t aoff[2][2], boff[2][2];
  int rowv[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q = (2 * w + i) * 8 + (lane >> 3);
      const int j = j0 + (q >> 6) * 128 + (q & 63) + h * 64;
      rowv[h][i] = j < n ? j : j0;
    }
  if (ids) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i) rowv[h][i] = ids[rowv[h][i]];
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      int64_t row = rowv[h][i];
      row = row < 0 ? 0 : (row >= V ? V - 1 : row);
      aoff[h][i] = (uint32_t)(row * d * 2 + pc * 16);
      const int q = (2 * w + i) * 8 + (lane >> 3);
      int m = m0 + (q >> 5) * 64 + (q & 31) + h * 32;
      m = m < M ? m : M - 1;
      boff[h][i] = (uint32_t)((int64_t)m * d * 2 + pc * 16);
    }
  const int nk = d / 64;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  auto fetch_a = [&](int st, int h) {
    const int c = st < nk ? st : nk - 1;
    const char* base = reinterpret_cast<const char*>(W) + (int64_t)c * 128;
    const uint32_t l = lds0 + (st & 1) * kGemmStage + h * 16384 + w * 2048;
    lds_fetch16(l, base, aoff[h][0]);
    lds_fetch16(l + 1024, base, aoff[h][1]);
  };
  auto fetch_b = [&](int st, int h) {
    const int c = st < nk ? st : nk - 1;
    const char* base = reinterpret_cast<const char*>(H) + (int64_t)c * 128;
    const uint32_t l = lds0 + (st & 1) * kGemmStage + 32768 + h * 16384 + w * 2048;
    lds_fetch16(l, base, boff[h][0]);
    lds_fetch16(l + 1024, base, boff[h][1]);
  };

  f32x4 acc[8][4];
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  // fragment addresses inside a half: row r (lane & 15 within the fragment), piece (lane >> 4) + 4 * kk, swizzled by r & 7
  const int fr = lane & 15, s7 = lane & 7;
  const uint32_t f0 = fr * 128 + (((lane >> 4)) ^ s7) * 16, f1 = fr * 128 + (((lane >> 4) + 4) ^ s7) * 16;
  bf16x8 af[4][2], b0[2][2], b1[2][2], b2[2][2];
  auto read_a = [&](int st, int h) {
    const char* p = smem + (st & 1) * kGemmStage + h * 16384 + wr * 8192;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      af[a][0] = *reinterpret_cast<const bf16x8*>(p + a * 2048 + f0);
      af[a][1] = *reinterpret_cast<const bf16x8*>(p + a * 2048 + f1);
    }
  };
  auto read_b = [&](int st, int h, bf16x8(&bq)[2][2]) {
    const char* p = smem + (st & 1) * kGemmStage + 32768 + h * 16384 + wh * 4096;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      bq[b][0] = *reinterpret_cast<const bf16x8*>(p + b * 2048 + f0);
      bq[b][1] = *reinterpret_cast<const bf16x8*>(p + b * 2048 + f1);
    }
  };
#define NS_COMPUTE(A0, B0, bq)                                                                                                          \
  do {                                                                                                                                  \
    __builtin_amdgcn_s_setprio(1);                                                                                                      \
    _Pragma("unroll") for (int kk = 0; kk < 2; ++kk) _Pragma("unroll") for (int a = 0; a < 4; ++a) _Pragma("unroll") for (int b = 0; b < 2; ++b) \
        acc[A0 + a][B0 + b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a][kk], bq[b][kk], acc[A0 + a][B0 + b], 0, 0, 0);             \
    __builtin_amdgcn_s_setprio(0);                                                                                                      \
  } while (0)

  // prologue
  fetch_a(0, 0);
  fetch_b(0, 0);
  fetch_b(0, 1);
  fetch_a(0, 1);
  fetch_a(1, 0);
  fetch_b(1, 0);
  fetch_b(1, 1);
  NS_WAIT_VM(10);
  NS_BARRIER();
  read_b(0, 0, b0);
  if (wr == 1) NS_BARRIER();                               // the second four wavefronts run one cluster behind the first
  auto step = [&](int st, bf16x8(&bc)[2][2], bf16x8(&bn)[2][2]) {
    read_a(st, 0);
    fetch_a(st + 1, 1);
    NS_WAIT_VM(10);
    NS_BARRIER();
    NS_COMPUTE(0, 0, bc);
    NS_BARRIER();
    read_b(st, 1, b1);
    NS_WAIT_VM(8);
    NS_BARRIER();
    NS_COMPUTE(0, 2, b1);
    NS_BARRIER();
    read_a(st, 1);
    fetch_a(st + 2, 0);
    fetch_b(st + 2, 0);
    NS_WAIT_VM(8);
    NS_BARRIER();
    NS_COMPUTE(4, 2, b1);
    NS_BARRIER();
    read_b(st + 1, 0, bn);
    fetch_b(st + 2, 1);
    NS_BARRIER();
    NS_COMPUTE(4, 0, bc);
    NS_BARRIER();
  };
  int st = 0;
  for (; st + 1 < nk; st += 2) {
    step(st, b0, b2);
    step(st + 1, b2, b0);
  }
  if (st < nk) step(st, b0, b2);
  if (wr == 0) NS_BARRIER();
  NS_WAIT_VM(0);                                           // the re-fetched last steps have landed before this LDS can be another workgroup's

#pragma unroll
  for (int a = 0; a < 8; ++a) {
    const int j = j0 + wr * 128 + a * 16 + 4 * (lane >> 4);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int m = m0 + wh * 64 + b * 16 + (lane & 15);
      if (m >= M || j >= n) continue;
      float* rowp = logits + (int64_t)m * ld;
      if (opos) {
        const int4 jo4 = j + 3 < opos_len ? *reinterpret_cast<const int4*>(opos + j) : make_int4(-1, -1, -1, -1);
        const int jo[4] = {jo4.x, jo4.y, jo4.z, jo4.w};
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (j + v < n && jo[v] >= 0) rowp[jo[v]] = acc[a][b][v];
      } else if (j + 3 < n) {
        *reinterpret_cast<f32x4_u*>(rowp + j) = acc[a][b];
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (j + v < n) rowp[j + v] = acc[a][b][v];
      }
    }
  }
}

static hipError_t run_gemm(const uint16_t* W, const uint16_t* H, const int32_t* ids, const int32_t* n_dev, int32_t n_fixed, int32_t cap_rows,
                           int32_t V, int32_t M, int32_t d, int64_t ld, float* logits, const int32_t* opos, hipStream_t s) {
  const int row_blocks = (cap_rows + 255) / 256, hid_blocks = (M + 255) / 256;
  const int64_t grid = (int64_t)((row_blocks + 7) / 8) * hid_blocks * 8;
  if (grid > 0x7fffffff || d % 64 != 0) return hipErrorInvalidValue;
  head_gemm_kernel<<<dim3((unsigned)grid), 512, 2 * kGemmStage, s>>>(W, H, ids, n_dev, n_fixed, V, M, d, ld, logits, row_blocks, hid_blocks, opos,
                                                                     cap_rows / 4 * 4);
  return hipGetLastError();
}

template <WideShape SHAPE>
static hipError_t configure_shared() {
  constexpr WideBlock b = kWideBlocks[SHAPE];
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(head_wide_shared_kernel<b.WR, b.WH, b.FR, b.FH, b.BK, b.D, false>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(head_wide_shared_kernel<b.WR, b.WH, b.FR, b.FH, b.BK, b.D, true>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
}

template <WideShape SHAPE>
static hipError_t configure_wide() {
  constexpr WideBlock b = kWideBlocks[SHAPE];
  const void* fns[] = {reinterpret_cast<const void*>(head_wide_kernel<b.WR, b.WH, b.FR, b.FH, b.BK, b.D, false>),
                       reinterpret_cast<const void*>(head_wide_kernel<b.WR, b.WH, b.FR, b.FH, b.BK, b.D, true>)};
  for (const void* f : fns) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t wide_configure_device() {
  hipError_t e = configure_wide<kWide32x16>();
  if (e == hipSuccess) e = configure_wide<kWide64x16>();
  if (e == hipSuccess) e = configure_wide<kWide32x32>();
  if (e == hipSuccess) e = configure_wide<kWide64x32>();
  if (e == hipSuccess) e = configure_wide<kWide32x64>();
  if (e == hipSuccess) e = configure_wide<kWide64x64>();
  if (e == hipSuccess) e = configure_wide<kWide128x64>();
  if (e == hipSuccess) e = configure_wide<kWide256x128>();
  if (e == hipSuccess) e = configure_wide<kWide256x256>();
  if (e == hipSuccess) e = configure_shared<kWide32x16>();
  if (e == hipSuccess) e = configure_shared<kWide32x32>();
  if (e == hipSuccess) e = configure_shared<kWide64x64>();
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(head_gemm_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  return e;
}

template <WideShape SHAPE, typename... A>
static hipError_t run_shape(A... a) {
  constexpr WideBlock b = kWideBlocks[SHAPE];
  return run_wide<b.WR, b.WH, b.FR, b.FH, b.BK, b.D>(a...);
}

template <typename... A>
static hipError_t run_wide_shape(WideShape shape, A... a) {
  switch (shape) {
    case kWide32x16: return run_shape<kWide32x16>(a...);
    case kWide64x16: return run_shape<kWide64x16>(a...);
    case kWide32x32: return run_shape<kWide32x32>(a...);
    case kWide64x32: return run_shape<kWide64x32>(a...);
    case kWide32x64: return run_shape<kWide32x64>(a...);
    case kWide64x64: return run_shape<kWide64x64>(a...);
    case kWide128x64: return run_shape<kWide128x64>(a...);
    case kWide256x128: return run_shape<kWide256x128>(a...);
    case kWide256x256: return run_shape<kWide256x256>(a...);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_head_wide(const void* W, const void* H, const int32_t* ids, const int32_t* n_dev, int32_t n_fixed, int32_t cap_rows,
                            int32_t V, int32_t batch, int32_t M, int32_t d, int64_t ld, int64_t ids_stride, float* logits,
                            const int32_t* opos, hipStream_t s) {
  const uint16_t* Wp = static_cast<const uint16_t*>(W);
  const uint16_t* Hp = static_cast<const uint16_t*>(H);
  const bool dense = n_dev == nullptr;
  const bool aligned = ((reinterpret_cast<uintptr_t>(W) | reinterpret_cast<uintptr_t>(H)) & 15) == 0;   // of the fetches into LDS
  const WideShape shape = wide_shape(M, d, batch, cap_rows, dense, aligned);
  if (shape == kWideGemm) return run_gemm(Wp, Hp, ids, n_dev, n_fixed, cap_rows, V, M, d, ld, logits, opos, s);
  return run_wide_shape(shape, Wp, Hp, ids, n_dev, n_fixed, cap_rows, V, batch, M, d, ld, ids_stride, logits, opos, 0,
                        (int)wide_by_die(M, batch, cap_rows, dense), s);
}

template <WideShape SHAPE, typename... A>
static hipError_t run_shared_shape(A... a) {
  constexpr WideBlock b = kWideBlocks[SHAPE];
  return run_wide_shared<b.WR, b.WH, b.FR, b.FH, b.BK, b.D>(a...);
}

hipError_t launch_head_wide_shared(const void* W, const void* H, const int32_t* ids, const int32_t* n_dev, int32_t cap_rows, int32_t V,
                                   int32_t rows_total, int32_t seq_rows, int32_t d, int64_t ld, float* logits, const int32_t* opos,
                                   int64_t opos_stride, hipStream_t s) {
  const uint16_t* Wp = static_cast<const uint16_t*>(W);
  const uint16_t* Hp = static_cast<const uint16_t*>(H);
  switch (wide_shared_shape(rows_total)) {
    case kWide32x16: return run_shared_shape<kWide32x16>(Wp, Hp, ids, n_dev, cap_rows, V, rows_total, d, ld, opos_stride, logits, opos, seq_rows, s);
    case kWide32x32: return run_shared_shape<kWide32x32>(Wp, Hp, ids, n_dev, cap_rows, V, rows_total, d, ld, opos_stride, logits, opos, seq_rows, s);
    default: return run_shared_shape<kWide64x64>(Wp, Hp, ids, n_dev, cap_rows, V, rows_total, d, ld, opos_stride, logits, opos, seq_rows, s);
  }
}

}  // namespace nanospec
