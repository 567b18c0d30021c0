// Eq. 1 on gathered rows for up to 16 hidden rows and many list rows: the hidden rows stay in registers, the list streams past them.
//
// The kernels of head.hip fetch the hidden rows again for every 16 list rows -- as many bytes out of L2 as the rows
// themselves at M = 16 -- and are launched over the capacity of the list.  Here the launch is as many workgroups as the chip
// holds, each takes an equal piece of the live rows, and a wavefront keeps its 1024 columns of all hidden rows (already in operand
// layout) for the whole piece.  What bounds it is HBM, and for sequences that share rows the bytes a die fetches beyond its L2 (64 of 2300 x
// 4096, M = 8: 0.6 GB, of which 0.38 are distinct rows).  Measured (before): 8400 x 8192, M = 16 29.7 us (37.8; a bare gather of the same rows 26.1), 32800 x 8192
// 100 us (107; 94.6), 30000 x 4096, M = 8 46 us (52; 42.2), 64 sequences of 2300 x 4096, M = 8 106 us (127), 32 58 us (73).
//
// Measured and not kept: quads dealt out in turn instead of contiguous pieces (the same time on lists, dense 189 to 212 us against 193); one step in flight
// (the same) or three and four (64 sequences 112 to 116 us: what is in flight then fills the die's L2); K-slices of 512 columns one after another with all
// sums kept in LDS, so that a die's L2 holds more rows at a time (64 sequences 103 us, 32 62); pieces cut at equal ids instead of equal counts
// (a tenth fewer bytes beyond L2, but the longest piece sets the time: 107 us).
#include "common.h"

namespace nanospec {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// sum over the four lanes of a quad, in every lane of it (DPP quad_perm: neighbours 1 apart, then 2 apart)
__device__ __forceinline__ float hold_quad_sum(float x) {
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xf, 0xf, true));   // quad_perm:[1,0,3,2]
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xf, 0xf, true));   // quad_perm:[2,3,0,1]
  return x;
}

// MT tiles of four hidden rows.  nw = blockDim.x / 64 wavefronts, wavefront w holds columns [1024 w, 1024 (w + 1)).  Operand layout of
// head_quad_kernel (head.hip): the 16 operand rows are 4 list rows x 4 column parts against 4 hidden rows x the same parts, so
// one load instruction covers 4 rows x 256 contiguous bytes.  A step is such a quad of list rows, eight loads a wavefront; the loads of
// two steps are in flight (128 KB on a compute unit with eight wavefronts), a step's registers are asked for again as soon as they are consumed.
// The products of a step are summed over the wavefronts at the end of a segment of at most `seg` rows, through LDS; a logit's sum has the same order wherever
// its row lies in the list.
// Piece p = die * parts + part of 8 * parts: consecutive workgroups go to the dies in turn, so that a die takes the same eighth of every
// sequence's list and finds the rows that sequences share in its own L2.
// TAIL: 1024 nw > d; pieces past column d are fetched from the row's start and zeroed.  LISTED: rows from ids, else 0 .. n - 1.
template <int MT, bool TAIL, bool LISTED>
__global__ __launch_bounds__(512, 2) void head_hold_kernel(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H,
                                                           const int32_t* __restrict__ ids, const int32_t* __restrict__ n_dev, int n_fixed,
                                                           int V, int batch, int M, int d, int64_t ld, int64_t ids_stride,
                                                           float* __restrict__ logits, int parts, int seg_max, const int32_t* __restrict__ opos) {
  constexpr int KS = 8, D = 2, MH = 4 * MT;
  extern __shared__ __attribute__((aligned(16))) float red[];             // [wavefront][hidden row][row of the segment], rows padded
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int orow = (lane & 15) >> 2, part = lane & 3, q = lane >> 4;      // operand row / column part / k group
  const int x = blockIdx.x & 7, xr = blockIdx.x >> 3;
  const int b = xr % batch, p = x * parts + xr / batch;
  const int n = n_dev ? n_dev[b] : n_fixed;
  const int col = w * (128 * KS) + q * 32 + part * 8;                     // + t * 128
  const u32x4 zero = u32x4{0u, 0u, 0u, 0u};

  // half of the hidden rows are asked for while the row count is on its way, the other half while the ids are
  const uint16_t* Hb = H + (int64_t)b * M * d;
  u32x4 hv[MT][KS];
  auto load_h = [&](int mt) {
    const int m = mt * 4 + orow;
    const uint16_t* hp = Hb + (int64_t)(m < M ? m : M - 1) * d;           // a row past M is a copy, never stored
#pragma unroll
    for (int t = 0; t < KS; ++t) hv[mt][t] = *reinterpret_cast<const u32x4*>(hp + (!TAIL || col + t * 128 < d ? col + t * 128 : 0));
  };
#pragma unroll
  for (int mt = 0; mt < MT / 2; ++mt) load_h(mt);

  const int np = 8 * parts, each = n / np, more = n - each * np;          // the first `more` pieces have a row more
  const int r0 = p * each + (p < more ? p : more), r1 = r0 + each + (p < more ? 1 : 0);
  if (r0 >= r1) return;
  if (LISTED) ids += b * ids_stride;
  if (opos) opos += b * ids_stride;
  logits += (int64_t)b * M * ld;
  const char* Wb = reinterpret_cast<const char*>(W);
  uint32_t pm[4];                                                         // masks of this lane's part: no branches around the sums over lanes
#pragma unroll
  for (int i = 0; i < 4; ++i) pm[i] = part == i ? 0xffffffffu : 0u;
  uint32_t okm = 0;
  if (TAIL) {
#pragma unroll
    for (int t = 0; t < KS; ++t) okm |= (col + t * 128 < d ? 1u : 0u) << t;
  }

  const int rows = r1 - r0, nseg = (rows + seg_max - 1) / seg_max;
  const int seg = ((rows + nseg - 1) / nseg + 3) & ~3, segp = seg_max + 4;
  for (int s0 = r0; s0 < r1; s0 += seg) {
    const int s1 = s0 + seg < r1 ? s0 + seg : r1, nq = (s1 - s0 + 3) >> 2;
    // list row of quad i for this lane; past the end the last row again
    auto id_of = [&](int i) {
      int j = s0 + i * 4 + orow;
      j = j < s1 ? j : s1 - 1;
      return LISTED ? ids[j] : j;
    };
    // a quad past the end: all lanes at one address
    auto fetch = [&](u32x4(&v)[KS], int id, int i) {
      id = id < 0 ? 0 : (id >= V ? V - 1 : id);
      const uint32_t row = (uint32_t)id * (uint32_t)(d * 2), c = (uint32_t)(w * (128 * KS) + (i < nq ? q * 32 + part * 8 : 0)) * 2;
#pragma unroll
      for (int t = 0; t < KS; ++t)
        v[t] = *reinterpret_cast<const u32x4*>(Wb + (TAIL ? row + ((okm >> t & 1) ? c + t * 256 : 0) : row + c + t * 256));
    };
    u32x4 wv[D][KS];
    int idn[D], id2[D];
#pragma unroll
    for (int i = 0; i < D; ++i) idn[i] = id_of(i);
#pragma unroll
    for (int i = 0; i < D; ++i) id2[i] = id_of(i + D);
    if (s0 == r0) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mt = MT / 2; mt < MT; ++mt) load_h(mt);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < D; ++i) {
      fetch(wv[i], idn[i], i);
      idn[i] = id2[i];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (TAIL && s0 == r0) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < KS; ++t) hv[mt][t] = (okm >> t & 1) ? hv[mt][t] : zero;
    }
    for (int i0 = 0; i0 < nq; i0 += D) {
#pragma unroll
      for (int u = 0; u < D; ++u) {
        const int i = i0 + u, id = idn[u];
        idn[u] = id_of(i + 2 * D);
        f32x4 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < KS; ++t) {
          u32x4 v = wv[u][t];
          if (TAIL) v = (okm >> t & 1) ? v : zero;
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, hv[mt][t]), acc[mt], 0, 0, 0);
        }
        fetch(wv[u], id, i + D);
        // result lane l holds product rows 4 * (l / 16) + v, column l % 16; the diagonal block entry is v == l % 4.  After the sum over
        // the parts all four lanes of a quad hold the logit of (list row q, hidden row 4 mt + orow): lane `part` keeps tile mt == part
        uint32_t y = 0;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const f32x4 a = acc[mt];
          const uint32_t s = (__float_as_uint(a[0]) & pm[0]) | (__float_as_uint(a[1]) & pm[1]) | (__float_as_uint(a[2]) & pm[2]) | (__float_as_uint(a[3]) & pm[3]);
          y |= __float_as_uint(hold_quad_sum(__uint_as_float(s))) & pm[mt];
        }
        if (part < MT && i < nq) red[(w * MH + part * 4 + orow) * segp + i * 4 + q] = __uint_as_float(y);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
    for (int m = w; m < M; m += nw)
      for (int j = lane; j < s1 - s0; j += 64) {
        float s = red[m * segp + j];
        for (int k = 1; k < nw; ++k) s += red[(k * MH + m) * segp + j];
        const int jo = opos ? opos[s0 + j] : s0 + j;                      // rows kept in an order of their own: column opos[j], nowhere if negative
        if (jo >= 0) logits[(int64_t)m * ld + jo] = s;
      }
    if (s1 < r1) __syncthreads();
  }
}

template <int MT>
static hipError_t run_hold(const uint16_t* W, const uint16_t* H, const int32_t* ids, const int32_t* n_dev, int32_t n_fixed, int32_t V, int32_t batch,
                           int32_t M, int32_t d, int64_t ld, int64_t ids_stride, float* logits, const int32_t* opos, HoldPlan h, hipStream_t s) {
  const unsigned grid = 8u * batch * h.parts, lds = (unsigned)hold_lds(h, M);
#define NS_HOLD(TAIL, LISTED)                                                                                                              \
  head_hold_kernel<MT, TAIL, LISTED><<<dim3(grid), 64 * h.NW, lds, s>>>(W, H, ids, n_dev, n_fixed, V, batch, M, d, ld, ids_stride, logits, \
                                                                        h.parts, h.seg, opos)
  if (d != 1024 * h.NW) {
    if (ids) NS_HOLD(true, true);
    else NS_HOLD(true, false);
  } else {
    if (ids) NS_HOLD(false, true);
    else NS_HOLD(false, false);
  }
#undef NS_HOLD
  return hipGetLastError();
}

hipError_t launch_head_hold(const void* W, const void* H, const int32_t* ids, const int32_t* n_dev, int32_t n_fixed, int32_t V,
                            int32_t batch, int32_t M, int32_t d, int64_t ld, int64_t ids_stride, float* logits, const int32_t* opos, hipStream_t s) {
  const uint16_t* Wp = static_cast<const uint16_t*>(W);
  const uint16_t* Hp = static_cast<const uint16_t*>(H);
  const HoldPlan h = hold_plan(d, batch, n_dev == nullptr);
  if (M <= 4) return run_hold<1>(Wp, Hp, ids, n_dev, n_fixed, V, batch, M, d, ld, ids_stride, logits, opos, h, s);
  if (M <= 8) return run_hold<2>(Wp, Hp, ids, n_dev, n_fixed, V, batch, M, d, ld, ids_stride, logits, opos, h, s);
  if (M <= 12) return run_hold<3>(Wp, Hp, ids, n_dev, n_fixed, V, batch, M, d, ld, ids_stride, logits, opos, h, s);
  return run_hold<4>(Wp, Hp, ids, n_dev, n_fixed, V, batch, M, d, ld, ids_stride, logits, opos, h, s);
}

template <int MT>
static hipError_t configure_hold() {
  const void* fns[] = {reinterpret_cast<const void*>(head_hold_kernel<MT, false, false>), reinterpret_cast<const void*>(head_hold_kernel<MT, false, true>),
                       reinterpret_cast<const void*>(head_hold_kernel<MT, true, false>), reinterpret_cast<const void*>(head_hold_kernel<MT, true, true>)};
  for (const void* f : fns) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t hold_configure_device() {
  hipError_t e = configure_hold<1>();
  if (e == hipSuccess) e = configure_hold<2>();
  if (e == hipSuccess) e = configure_hold<3>();
  if (e == hipSuccess) e = configure_hold<4>();
  return e;
}

}  // namespace nanospec
