// Eq. 1 on gathered rows for 17 to 64 hidden rows, K sliced over the wavefronts of a workgroup.
//
// head_wide_kernel (wide.hip) parks both operand blocks of a step in LDS and every wavefront multiplies its part of the block: each byte is
// written once and read by two to four wavefronts, 32 KB of LDS reads for 16 KB of operands with 32 x 32 blocks, and a step is a chain of a park, a barrier and the reads
// behind it -- 620 cycles for 16 KB a compute unit could take out of L2 in 256.  Here a wavefront multiplies the whole block over its own steps of 64 columns
// (w, w + 4, ...): every byte goes straight from memory into the wavefront's own ring of LDS slots and is read once, nobody waits for anybody until the
// sums of the four wavefronts are added in fixed order at the end.  A launch that fits the chip then takes about 5 us (launch, row count, ids and first rows one after the other, the sums) and the bytes a compute unit
// fetches, rows and hidden rows alike (93 GB/s each), so the pieces are equal: the live rows are dealt out over as many workgroups as the chip holds, in blocks of any multiple of
// 8 rows, and the block of hidden rows is what makes (rows + hidden rows) of a workgroup smallest (kslice_plan in choose.h).
// Measured (before): 3000 x 3584, M = 64 9.5 us (11.2), 1000 x 4096, M = 64 6.4 (9.5), 3000 x 4096, M = 40 9.8 (12.1), 8400 x 8192, M = 64 41.5 (62.5), 2000 out of 7000 x 4096, M = 24 7.4 (11.4),
// 8 sequences of 600 x 4096, M = 48 13.7 (19), 4 of 1500 out of 3000, M = 40 13.2 (16.2).
// Measured and not kept: eight wavefronts (the same); a ring half as deep and two workgroups per compute unit (8400 x 8192 43 us, 3000 x 3584 9.6, better only where pieces are several blocks: 20000 x 4096, M = 64
// 45 against 47); the width picked on the device by the row count, all of them in one kernel (0.3 to 1 us slower); row ids asked for before the row count has arrived (the same); 16 x 64 and 16 x 32 blocks (1.2 to 1.5 times).
#include "common.h"

namespace nanospec {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSliceWaves = 4;

// slots of a wavefront's ring, one step (8 rows of 128 bytes to the KB) of L KB to a slot
constexpr int slice_ring(int L) { return L <= 4 ? 4 : L <= 6 ? 3 : 2; }

// the wait behind lds_fetch16 (global_load_lds, common.h)
template <int N>
__device__ __forceinline__ void slice_wait() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// The block of list rows [j0, j1), at most 8 * LA, and hidden rows [m0, m0 + 8 * LB) below M.  A slot holds LA + LB KB: one instruction fetches 8 rows x 64 columns, the 16-byte pieces
// of a row permuted by the row's low three bits (the fetching lanes permute their addresses), so that the reads of a fragment -- 16 rows, one piece each -- meet no bank
// twice.  Rows past j1 are copies of the last one, hidden rows past M of row M - 1; with an odd LA (LB) the last fragment's second half is whatever lies behind (LDS
// allocated for it).  None of these is stored.
template <int LA, int LB>
__device__ __forceinline__ void slice_block(char* smem, const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, const int32_t* __restrict__ ids, int V, int M,
                                            int d, int64_t ld, float* __restrict__ logits, int j0, int j1, int m0, const int32_t* __restrict__ opos) {
  constexpr int NW = kSliceWaves, L = LA + LB, FR = (LA + 1) / 2, FH = (LB + 1) / 2, R = slice_ring(L), SLOT = L * 1024, JP = 16 * FR + 4;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pc = (lane & 7) ^ (lane >> 3);                              // row & 7 == lane >> 3 in every instruction: the permuted piece
  uint32_t aoff[LA], boff[LB];                                          // byte offsets of this lane's rows
  int rowv[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int j = j0 + i * 8 + (lane >> 3);
    rowv[i] = j < j1 ? j : j1 - 1;
  }
  if (ids) {
#pragma unroll
    for (int i = 0; i < LA; ++i) rowv[i] = ids[rowv[i]];
  }
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int row = rowv[i] < 0 ? 0 : (rowv[i] >= V ? V - 1 : rowv[i]);
    aoff[i] = (uint32_t)row * (uint32_t)(d * 2) + pc * 16;
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const int m = m0 + i * 8 + (lane >> 3);
    boff[i] = (uint32_t)(m < M ? m : M - 1) * (uint32_t)(d * 2) + pc * 16;
  }
  const int nk = (d + 63) / 64, mine = (nk - w + NW - 1) / NW;          // this wavefront's steps: w, w + 4, ...
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + w * (R * SLOT);
  const char* slots = smem + w * (R * SLOT);
  // own step i into slot r; the last step's columns past d: the row's start
  auto fetch = [&](int i, int r) {
    const int k0 = (w + i * NW) * 64;
    const uint32_t l = lds0 + r * SLOT;
    if (k0 + 64 <= d) {
      const char *wb = reinterpret_cast<const char*>(W) + (int64_t)k0 * 2, *hb = reinterpret_cast<const char*>(H) + (int64_t)k0 * 2;
#pragma unroll
      for (int q = 0; q < LB; ++q) lds_fetch16(l + (LA + q) * 1024, hb, boff[q]);
#pragma unroll
      for (int q = 0; q < LA; ++q) lds_fetch16(l + q * 1024, wb, aoff[q]);
    } else {
      const uint32_t co = k0 + pc * 8 < d ? k0 * 2 : (uint32_t)-pc * 16;   // offsets hold pc * 16
#pragma unroll
      for (int q = 0; q < LB; ++q) lds_fetch16(l + (LA + q) * 1024, H, boff[q] + co);
#pragma unroll
      for (int q = 0; q < LA; ++q) lds_fetch16(l + q * 1024, W, aoff[q] + co);
    }
  };
#pragma unroll
  for (int q = 0; q < R; ++q)
    if (q < mine) fetch(q, q);
  f32x4 acc[FR][FH];
#pragma unroll
  for (int a = 0; a < FR; ++a)
#pragma unroll
    for (int c = 0; c < FH; ++c) acc[a][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  // fragment addresses inside a slot: row lane & 15, piece (lane >> 4) + 4 * kk, permuted by row & 7
  const int fr = lane & 15, s7 = lane & 7;
  const uint32_t f[2] = {(uint32_t)(fr * 128 + ((lane >> 4) ^ s7) * 16), (uint32_t)(fr * 128 + (((lane >> 4) + 4) ^ s7) * 16)};
  int r = 0;
  for (int i = 0; i < mine; ++i) {
    if (i + R <= mine) slice_wait<(R - 1) * L>();                       // this slot's fetches have landed, the younger slots' are in flight
    else slice_wait<0>();                                               // the last steps: fewer are in flight
    __builtin_amdgcn_sched_barrier(0);
    const char* s = slots + r * SLOT;
    bf16x8 af[FR][2], bq[FH][2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int a = 0; a < FR; ++a) af[a][kk] = *reinterpret_cast<const bf16x8*>(s + a * 2048 + f[kk]);
#pragma unroll
      for (int c = 0; c < FH; ++c) bq[c][kk] = *reinterpret_cast<const bf16x8*>(s + LA * 1024 + c * 2048 + f[kk]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                  // the fragments are in registers: the slot can be refilled
    __builtin_amdgcn_sched_barrier(0);
    if (i + R < mine) fetch(i + R, r);
    __builtin_amdgcn_sched_barrier(0);
    const int k0 = (w + i * NW) * 64;
    if (k0 + 64 > d) {                                                  // uniform: the last step of a d that is no multiple of 64, columns past d are zeros on both sides
      const bf16x8 zero = __builtin_bit_cast(bf16x8, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bool in = k0 + ((lane >> 4) + 4 * kk) * 8 < d;
#pragma unroll
        for (int a = 0; a < FR; ++a) af[a][kk] = in ? af[a][kk] : zero;
#pragma unroll
        for (int c = 0; c < FH; ++c) bq[c][kk] = in ? bq[c][kk] : zero;
      }
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int a = 0; a < FR; ++a)
#pragma unroll
        for (int c = 0; c < FH; ++c) acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a][kk], bq[c][kk], acc[a][c], 0, 0, 0);
    r = r + 1 == R ? 0 : r + 1;
  }
  __syncthreads();                                                      // all fetches have landed, all fragments are read: this LDS takes the sums
  // lane l holds list rows 4 * (l / 16) + v of hidden row l % 16 of a fragment
  float* red = reinterpret_cast<float*>(smem) + w * (16 * FH * JP);     // [hidden row][list row]
#pragma unroll
  for (int a = 0; a < FR; ++a)
#pragma unroll
    for (int c = 0; c < FH; ++c) *reinterpret_cast<f32x4*>(red + (c * 16 + (lane & 15)) * JP + a * 16 + 4 * (lane >> 4)) = acc[a][c];
  __syncthreads();
  const float* sum = reinterpret_cast<const float*>(smem);
  for (int o = threadIdx.x; o < 64 * LA * LB; o += 64 * NW) {           // one logit at a time: four with 16-byte reads and stores 0.4 us more at 1000 rows
    const int c = o / (8 * LA), j = o % (8 * LA), m = m0 + c;
    if (m >= M || j0 + j >= j1) continue;
    float v = sum[c * JP + j];
#pragma unroll
    for (int k = 1; k < NW; ++k) v += sum[(k * 16 * FH + c) * JP + j];
    const int jo = opos ? opos[j0 + j] : j0 + j;                        // rows kept in an order of their own: column opos[j], nowhere if negative
    if (jo >= 0) logits[(int64_t)m * ld + jo] = v;
  }
}

// n / by for n * by below 2^32, from 2^32 / by rounded up; by == 1 has no such reciprocal (0)
__device__ __forceinline__ uint32_t slice_over(uint32_t n, uint32_t over) { return over ? __umulhi(n, over) : n; }

// Grid: 8 * parts pieces of every sequence's list times hid_blocks.  Piece p = die * parts + part (consecutive workgroups go to the dies in turn): a die takes the same
// eighth of every list, and the workgroups that share a piece's rows run on it one behind the other.  Quotients by the plan's numbers are products with the host's reciprocals: a
// division in the way of the first fetch takes longer than the rest of this.
template <int LB>
__global__ __launch_bounds__(64 * kSliceWaves, 2) void head_kslice_kernel(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H,
                                                                          const int32_t* __restrict__ ids, const int32_t* __restrict__ n_dev, int V,
                                                                          int batch, int M, int d, int64_t ld, int64_t ids_stride, float* __restrict__ logits,
                                                                          SlicePlan plan, const int32_t* __restrict__ opos) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const uint32_t x = blockIdx.x & 7, xr = blockIdx.x >> 3, y = slice_over(xr, plan.over_hid), hb = xr - y * plan.hid_blocks, part = slice_over(y, plan.over_batch), b = y - part * batch;
  const int n = n_dev[b];
  const int np = 8 * plan.parts, p = x * plan.parts + part, each = slice_over(n, plan.over_pieces), more = n - each * np;   // the first `more` pieces have a row more
  const int r0 = p * each + (p < more ? p : more), r1 = r0 + each + (p < more ? 1 : 0);
  if (r0 >= r1) return;
  if (ids) ids += b * ids_stride;
  if (opos) opos += b * ids_stride;
  H += (int64_t)b * M * d;
  logits += (int64_t)b * M * ld;
  const int m0 = hb * 8 * LB;
  int seg = r1 - r0;
  if (seg > plan.rows) {
    const int nseg = (seg + plan.rows - 1) / plan.rows;
    seg = (seg + nseg - 1) / nseg;
  }
  for (int j0 = r0; j0 < r1; j0 += seg) {
    const int j1 = j0 + seg < r1 ? j0 + seg : r1;
    if (j0 != r0) __syncthreads();                                      // the sums have been read
    switch ((j1 - j0 + 7) / 8) {
      case 1: slice_block<1, LB>(smem, W, H, ids, V, M, d, ld, logits, j0, j1, m0, opos); break;
      case 2: slice_block<2, LB>(smem, W, H, ids, V, M, d, ld, logits, j0, j1, m0, opos); break;
      case 3: slice_block<3, LB>(smem, W, H, ids, V, M, d, ld, logits, j0, j1, m0, opos); break;
      case 4: slice_block<4, LB>(smem, W, H, ids, V, M, d, ld, logits, j0, j1, m0, opos); break;
      case 5: slice_block<5, LB>(smem, W, H, ids, V, M, d, ld, logits, j0, j1, m0, opos); break;
      case 6: slice_block<6, LB>(smem, W, H, ids, V, M, d, ld, logits, j0, j1, m0, opos); break;
      default: slice_block<8, LB>(smem, W, H, ids, V, M, d, ld, logits, j0, j1, m0, opos); break;
    }
  }
}

// dynamic LDS for blocks of up to `rows` list rows and 8 * LB hidden rows: four rings and half a fragment behind the last, or the sums
constexpr int slice_lds(int LB, int rows) {
  int most = 0;
  for (int LA = 1; 8 * LA <= rows; ++LA) {
    if (LA == 7) continue;
    const int L = LA + LB, rings = kSliceWaves * slice_ring(L) * L * 1024 + 1024, sums = kSliceWaves * 16 * ((LB + 1) / 2) * (16 * ((LA + 1) / 2) + 4) * 4;
    most = rings > most ? rings : most;
    most = sums > most ? sums : most;
  }
  return most;
}
static_assert(slice_lds(8, 64) <= 160 * 1024 && slice_lds(2, 64) <= 160 * 1024, "LDS of a compute unit");

template <int LB>
static hipError_t run_kslice(const void* W, const void* H, const int32_t* ids, const int32_t* n_dev, int32_t V, int32_t batch, int32_t M, int32_t d, int64_t ld,
                             int64_t ids_stride, float* logits, const int32_t* opos, const SlicePlan& p, hipStream_t s) {
  head_kslice_kernel<LB><<<dim3(8u * p.parts * p.hid_blocks * batch), 64 * kSliceWaves, slice_lds(LB, p.rows), s>>>(
      static_cast<const uint16_t*>(W), static_cast<const uint16_t*>(H), ids, n_dev, V, batch, M, d, ld, ids_stride, logits, p, opos);
  return hipGetLastError();
}

hipError_t launch_head_kslice(const void* W, const void* H, const int32_t* ids, const int32_t* n_dev, int32_t cap_rows, int32_t V, int32_t batch, int32_t M,
                              int32_t d, int64_t ld, int64_t ids_stride, float* logits, const int32_t* opos, hipStream_t s) {
  const SlicePlan p = kslice_plan(M, batch, cap_rows);
  switch (p.LB) {
    case 2: return run_kslice<2>(W, H, ids, n_dev, V, batch, M, d, ld, ids_stride, logits, opos, p, s);
    case 3: return run_kslice<3>(W, H, ids, n_dev, V, batch, M, d, ld, ids_stride, logits, opos, p, s);
    case 4: return run_kslice<4>(W, H, ids, n_dev, V, batch, M, d, ld, ids_stride, logits, opos, p, s);
    case 5: return run_kslice<5>(W, H, ids, n_dev, V, batch, M, d, ld, ids_stride, logits, opos, p, s);
    case 6: return run_kslice<6>(W, H, ids, n_dev, V, batch, M, d, ld, ids_stride, logits, opos, p, s);
    default: return run_kslice<8>(W, H, ids, n_dev, V, batch, M, d, ld, ids_stride, logits, opos, p, s);
  }
}

template <int LB>
static hipError_t configure_kslice() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(head_kslice_kernel<LB>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
}

hipError_t kslice_configure_device() {
  hipError_t e = configure_kslice<2>();
  if (e == hipSuccess) e = configure_kslice<3>();
  if (e == hipSuccess) e = configure_kslice<4>();
  if (e == hipSuccess) e = configure_kslice<5>();
  if (e == hipSuccess) e = configure_kslice<6>();
  if (e == hipSuccess) e = configure_kslice<8>();
  return e;
}

}  // namespace nanospec
