// Draft-token selection (paper Alg. 1, SelectDraftTokens(z', I); operator T_K of Sec. 3.2):
// the k largest logits of every row, ordered by value descending then global id ascending, mapped
// from the position in the active list back to the global token id.
//
// Every lane keeps a run of consecutive logits in registers, so "lower position" means "lower lane,
// then lower register".  A wavefront extracts its k best in k rounds: a DPP max-reduction of the
// lane maxima, a ballot of the lanes that hold that maximum (the lowest such lane owns the
// lowest-position occurrence), one readlane for the register index, and the winner is blanked.
// The wavefronts' winners meet in LDS in position order and one wavefront repeats the rounds over
// them.  Few rows longer than one workgroup reaches are cut into chunks whose winners a second kernel
// ranks.  Values of -inf mark "nothing left" (logits are finite by contract).
//
// Fast path in front of the rounds: lane l of wavefront w always holds positions (64w + l)*EPT ..., whatever
// the row's length n, so the logits are requested before n has arrived and masked afterwards.  The nwe
// wavefronts that are at least half full (or the first one) each report their ceil(k/nwe)-th largest lane
// maximum; the smallest report is a lower bound T on the row's k-th largest value (at least k lanes hold
// something >= T), so only elements >= T can be winners.  They are compacted in position order into LDS
// (typically one or two dozen; a DPP prefix sum over the lanes and one over the wavefront totals), every
// thread ranks one candidate against all others while its global id is being fetched, and rank r < k is
// output slot r.  If more than kCandMax elements survive (heavy ties) the kernel falls back to the rounds.
// Measured and not kept: handing out the LDS slots with one atomic counter and breaking ties by position;
// splitting the valid runs evenly over the wavefronts (the layout then depends on n: c2 4.2 against
// 4.1 us, c3 5.0 against 4.6); fetching every lane's 16 ids beside its logits so that the winners' ids
// need no second round trip (4.3-4.4 us on c2); a single-pass threshold -- the smallest maximum of the filled
// 16-lane rows, no rounds -- which lets so many more candidates through that nothing is gained at 3k
// elements (3.74 against 3.72 us) and the 8k-element case falls back to the rounds (12.0 against 6.6 us).
// Half-wavefronts as voters (twice the voters, half the rounds, two thresholds per round) helped only
// the unlucky lengths with a single voting wavefront (1.3k elements: 4.0 against 4.3 us) and cost 0.1-1 us elsewhere.
//
// LSE variants (Sec. 4.2: the draft distribution is the softmax renormalised over the active set):
// the same selection, with the values written as log-probabilities z - log(sum_i exp z_i), i over the
// row's n entries.  The row maximum falls out of the first threshold round, the sum of exp(z - max)
// is taken wavefront by wavefront and added in wavefront order (chunk order in the merge kernel), so
// the result does not depend on timing.
#include <limits.h>

#include "common.h"

namespace nanospec {

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_max(float x) {
  const int ninf = __float_as_int(-INFINITY);
  const int y = __builtin_amdgcn_update_dpp(ninf, __float_as_int(x), CTRL, ROW_MASK, 0xf, false);
  return fmaxf(x, __int_as_float(y));
}

// maximum over the 64 lanes, returned in every lane

__device__ __forceinline__ float wave_max(float x) {
  x = dpp_max<0x111, 0xf>(x);   // row_shr:1
  x = dpp_max<0x112, 0xf>(x);   // row_shr:2
  x = dpp_max<0x114, 0xf>(x);   // row_shr:4
  x = dpp_max<0x118, 0xf>(x);   // row_shr:8   -> lane 15 of each row holds the row maximum
  x = dpp_max<0x142, 0xa>(x);   // row_bcast:15 into rows 1 and 3
  x = dpp_max<0x143, 0xc>(x);   // row_bcast:31 into rows 2 and 3 -> lane 63 holds the maximum
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add(float x) {
  const int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROW_MASK, 0xf, false);
  return x + __int_as_float(y);
}

// sum over the 64 lanes in a fixed order, returned in every lane
__device__ __forceinline__ float wave_add(float x) {
  x = dpp_add<0x111, 0xf>(x);
  x = dpp_add<0x112, 0xf>(x);
  x = dpp_add<0x114, 0xf>(x);
  x = dpp_add<0x118, 0xf>(x);
  x = dpp_add<0x142, 0xa>(x);
  x = dpp_add<0x143, 0xc>(x);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// v[e] for a lane-varying e in [0, 16): a select tree (4 compares + 15 selects) instead of 16 predicated
// moves.  The elements arrive as sixteen scalars: selects between array elements get folded into a
// lane-varying array index, and that puts the whole array into scratch memory.
__device__ __forceinline__ float sel(bool c, float a, float b) { return c ? a : b; }
__device__ __forceinline__ float pick16(float v0, float v1, float v2, float v3, float v4, float v5, float v6, float v7,
                                        float v8, float v9, float v10, float v11, float v12, float v13, float v14,
                                        float v15, int e) {
  const bool b0 = e & 1, b1 = e & 2, b2 = e & 4, b3 = e & 8;
  const float a0 = sel(b0, v1, v0), a1 = sel(b0, v3, v2), a2 = sel(b0, v5, v4), a3 = sel(b0, v7, v6);
  const float a4 = sel(b0, v9, v8), a5 = sel(b0, v11, v10), a6 = sel(b0, v13, v12), a7 = sel(b0, v15, v14);
  const float c0 = sel(b1, a1, a0), c1 = sel(b1, a3, a2), c2 = sel(b1, a5, a4), c3 = sel(b1, a7, a6);
  return sel(b3, sel(b2, c3, c2), sel(b2, c1, c0));
}

// k rounds over the EPT values each lane holds (position = lane*EPT + register index).
// emit(r, value, position) is called by every lane with wave-uniform arguments; value == -inf
// means that fewer than r+1 elements exist.
template <int EPT, typename Emit>
__device__ __forceinline__ void wave_select(float (&v)[EPT], int k, int lane, Emit emit) {
  for (int r = 0; r < k; ++r) {
    float ml = v[0];
#pragma unroll
    for (int e = 1; e < EPT; ++e) ml = fmaxf(ml, v[e]);
    const float m = wave_max(ml);
    const unsigned long long ball = __ballot(ml == m);
    const int L = ball ? __ffsll(ball) - 1 : 0;
    int ef = 0;
#pragma unroll
    for (int e = EPT - 1; e >= 0; --e) ef = (v[e] == m) ? e : ef;
    const int eL = __builtin_amdgcn_readlane(ef, L);
    emit(r, ball ? m : -INFINITY, L * EPT + eL);
    const bool mine = lane == L;
#pragma unroll
    for (int e = 0; e < EPT; ++e) v[e] = (mine && e == eL) ? -INFINITY : v[e];
  }
}

// One workgroup of NW wavefronts selects the k best of elements [c*CH, (c+1)*CH) of row (b, m),
// CH = NW*64*EPT.  FINAL: write global ids / values; else (value, position) for the merge kernel --
// unless the whole row fits the first chunk (n <= CH, known only on the device): then chunk 0 writes the
// final result itself, the other chunks leave at once and the merge kernel has nothing to do.
constexpr int kLaneCand = 4;   // candidates per lane the owner path keeps in registers

template <int EPT, int NW, bool FINAL, bool LSE>
__device__ __forceinline__ void topk_select(const float* __restrict__ logits, int64_t ld, const int32_t* __restrict__ ids, int64_t ids_stride,
                                            const int32_t* __restrict__ n_dev, int n_fixed, int M, int k, int32_t* __restrict__ out_ids,
                                            float* __restrict__ out_vals, float* __restrict__ cand_val, int32_t* __restrict__ cand_pos,
                                            float2* __restrict__ cand_ms) {
  constexpr int E2 = (NW * kMaxK + 63) / 64;
  __shared__ float s_val[NW * kMaxK];
  __shared__ int s_pos[NW * kMaxK];
  const int c = blockIdx.x, m = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row = (int64_t)b * M + m;
  const float* src = logits + row * ld;
  // Position order is (wavefront, lane, register) and does not depend on the row's length, so the logits
  // are requested before the length has arrived: bounded by the row stride, masked by n afterwards.
  const int cbase = c * (NW * 64 * EPT);
  const int p0 = cbase + (wave * 64 + lane) * EPT;         // first position of this lane's run
  float v[EPT];
  if ((ld & 3) == 0) {
#pragma unroll
    for (int e = 0; e < EPT; e += 4) {
      float4 x = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      if (p0 + e < ld) x = *reinterpret_cast<const float4*>(src + p0 + e);   // row stride is a multiple of 4
      v[e] = x.x;
      v[e + 1] = x.y;
      v[e + 2] = x.z;
      v[e + 3] = x.w;
    }
  } else {
    // rows at any 4-byte address: one 16-byte load more from the aligned address below the run, shifted into place (16 single
    // loads per lane, 64 bytes apart, took twice the time: 60 rows of 30001 18 against 10 us); the pieces that reach over the row's ends are read element by element
    const int sh = (int)(((uint32_t)reinterpret_cast<uintptr_t>(src) & 15u) >> 2);   // uniform: elements from that address to the run
    float w[EPT + 4];
#pragma unroll
    for (int e = 0; e < EPT + 4; e += 4) {
      const int q = p0 - sh + e;
      float4 x = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      if (q >= 0 && q + 3 < ld) {
        x = *reinterpret_cast<const float4*>(src + q);
      } else if (q + 3 >= 0 && q < ld) {
        if (q >= 0) x.x = src[q];
        if (q + 1 >= 0 && q + 1 < ld) x.y = src[q + 1];
        if (q + 2 >= 0 && q + 2 < ld) x.z = src[q + 2];
        if (q + 3 < ld) x.w = src[q + 3];
      }
      w[e] = x.x;
      w[e + 1] = x.y;
      w[e + 2] = x.z;
      w[e + 3] = x.w;
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) v[e] = sel(sh & 2, sel(sh & 1, w[e + 3], w[e + 2]), sel(sh & 1, w[e + 1], w[e]));
  }
  const int n = n_dev ? n_dev[b] : n_fixed;
#pragma unroll
  for (int e = 0; e < EPT; ++e) v[e] = (p0 + e < n) ? v[e] : -INFINITY;
  // Wavefronts that are at least half full (or the first one) vote on the threshold; nwa hold anything at all.
  const int left = n - cbase;
  const int runs = left > 0 ? (left + EPT - 1) / EPT : 0;
  int nwe = (runs + 32) / 64;
  nwe = nwe < 1 ? 1 : (nwe > NW ? NW : nwe);
  int nwa = (runs + 63) / 64;
  nwa = nwa > NW ? NW : nwa;
  const bool fin = FINAL || n <= NW * 64 * EPT;           // uniform over the grid row
  if (!FINAL && fin && c != 0) return;
  float lse = 0.f;                                        // log sum exp of the row (LSE && fin)
  __shared__ float s_thr[NW];
  __shared__ float s_wmax[NW];
  __shared__ float s_sum[NW];
  __shared__ int s_cnt[NW];
  // A wavefront that holds nothing of the row leaves at once (a barrier waits only for the wavefronts that
  // are still running): with sixteen wavefronts on four SIMDs every instruction of an idle one delays the
  // others.  It first leaves the neutral entries the others will read; the first four always stay, for the
  // per-thread chores below (up to kCandMax candidates, k padding slots).
  const int nwl = nwa > 4 ? nwa : (NW < 4 ? NW : 4);      // wavefronts that stay, 0 .. nwl-1
  if (wave >= nwl) {
    if (lane == 0) {
      s_cnt[wave] = 0;
      s_wmax[wave] = -INFINITY;
      s_sum[wave] = 0.f;
    }
    if (lane < k) s_val[wave * k + lane] = -INFINITY;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the entries are in LDS before this wavefront is gone
    return;
  }
  // ---- fast path: threshold from lane maxima, compaction, ranking
  {
    __shared__ __attribute__((aligned(16))) float s_cv[kCandMax + 4];
    __shared__ int s_cp[kCandMax];
    float ml = v[0];
#pragma unroll
    for (int e = 1; e < EPT; ++e) ml = fmaxf(ml, v[e]);
    float x = ml, thr = -INFINITY;
    const int rounds = (k + nwe - 1) / nwe;                // nwe * rounds >= k lanes hold something >= T
    float wmax = -INFINITY, wsum = 0.f;
    for (int r = 0; r < rounds; ++r) {
      thr = wave_max(x);
      if (LSE && r == 0 && wave < nwa) {                    // the first round's result is the wavefront's maximum;
        wmax = thr;                                         // its exp-sum is independent work between the rounds
        const float ref = wmax == -INFINITY ? 0.f : wmax;   // nothing valid here: every term is exp(-inf) = 0
        float se = 0.f;
#pragma unroll
        for (int e = 0; e < EPT; ++e) se += __expf(v[e] - ref);
        wsum = wave_add(se);
      }
      const unsigned long long ball = __ballot(x == thr);
      const int L = ball ? __ffsll(ball) - 1 : 0;
      if (lane == L) x = -INFINITY;
    }
    if (lane == 0) {
      s_thr[wave] = thr;
      if (LSE) {
        s_wmax[wave] = wmax;
        s_sum[wave] = wsum;
      }
    }
    __syncthreads();
    float T = s_thr[0];
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) T = fminf(T, ww < nwe ? s_thr[ww] : INFINITY);
    if (LSE) {                                              // wavefront (max, sum) pairs -> the row's, in wavefront order
      const float wm = lane < NW ? s_wmax[lane] : -INFINITY;   // lane ww holds wavefront ww's pair
      float zmax = wave_max(wm);
      zmax = zmax == -INFINITY ? 0.f : zmax;                // empty chunk: every factor below is exp(-inf) = 0
      const float se = wave_add(lane < NW ? s_sum[lane] * expf(wm - zmax) : 0.f);
      if (fin) lse = zmax + logf(se);
      else if (tid == 0) cand_ms[row * gridDim.x + c] = make_float2(zmax, se);
    }
    uint32_t flags = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) flags |= (uint32_t)((p0 + e < n) && (v[e] >= T)) << e;
    const int mine = __popc(flags);
    int incl = mine;                                      // inclusive prefix sum over the lanes, by DPP
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, false);   // row_shr:1
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, false);   // row_shr:2
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, false);   // row_shr:4
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, false);   // row_shr:8
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    const int crowded = __ballot(mine > kLaneCand) != 0ull ? 1 << 20 : 0;   // some lane holds more than the owner path keeps
    if (lane == 63) s_cnt[wave] = incl | crowded;
    __syncthreads();
    int off = incl - mine, C = 0, any_crowded = 0;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      const int t = s_cnt[ww] & 0xfffff;
      any_crowded |= s_cnt[ww] >> 20;
      if (ww < wave) off += t;
      C += t;
    }
    if (EPT == 16 && C <= kCandMax && !any_crowded) {     // uniform over the workgroup
      // Owner path: the lane that holds a candidate asks for its global id at once (up to kLaneCand per
      // lane), the values alone meet in LDS, every thread ranks one of them, and the owner -- whose id has
      // arrived meanwhile -- writes the output slot its candidate's rank names.
      float cval[kLaneCand];
      int cgid[kLaneCand];
      uint32_t f = flags;
#pragma unroll
      for (int j = 0; j < kLaneCand; ++j) {
        cval[j] = 0.f;
        cgid[j] = 0;
        if (__ballot(f != 0u) != 0ull) {                    // some lane of this wavefront has a j-th candidate
          const int e = f ? __ffs(f) - 1 : 0;
          cval[j] = pick16(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10], v[11], v[12], v[13], v[14],
                           v[15], e);
          cgid[j] = p0 + e;
          if (f) {
            if (fin && ids) cgid[j] = ids[b * ids_stride + p0 + e];
            s_cv[off + j] = cval[j];
          }
          f &= f - 1u;
        }
      }
      if (tid < 4) s_cv[C + tid] = __builtin_nanf("");     // pads the last group of four; compares false with everything
      if (tid < C) s_cp[tid] = 0;                           // rank of candidate tid, accumulated below
      __syncthreads();
      // Work item (t, g): candidate t against the g-th group of four candidates; t is the fast index
      // (padded to a power of two), so a few dozen candidates are ranked in one sweep of the workgroup.
      const int lg = C <= 1 ? 0 : 32 - __clz(C - 1);
      const int items = ((C + 3) >> 2) << lg;
      for (int w = tid; w < items; w += 64 * nwl) {
        const int t = w & ((1 << lg) - 1), q = (w >> lg) * 4;
        if (t < C) {
          const float val = s_cv[t];
          const float4 o = *reinterpret_cast<const float4*>(&s_cv[q]);
          int r = (o.x > val || (o.x == val && q < t)) ? 1 : 0;         // list order is position order
          r += (o.y > val || (o.y == val && q + 1 < t)) ? 1 : 0;
          r += (o.z > val || (o.z == val && q + 2 < t)) ? 1 : 0;
          r += (o.w > val || (o.w == val && q + 3 < t)) ? 1 : 0;
          if (r) atomicAdd(&s_cp[t], r);
        }
      }
      if (tid >= C && tid < k) {                            // padding slots when fewer than k exist
        if (fin) {
          out_ids[row * k + tid] = -1;
          if (out_vals) out_vals[row * k + tid] = -INFINITY;
        } else {
          cand_val[(row * gridDim.x + c) * k + tid] = -INFINITY;
          cand_pos[(row * gridDim.x + c) * k + tid] = -1;
        }
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < kLaneCand; ++j) {
        const int rank = j < mine ? s_cp[off + j] : k;
        if (rank < k) {
          if (fin) {
            const int64_t o = row * k + rank;
            out_ids[o] = cgid[j];
            if (out_vals) out_vals[o] = (LSE && cval[j] != -INFINITY) ? cval[j] - lse : cval[j];
          } else {
            const int64_t o = (row * gridDim.x + c) * k + rank;
            cand_val[o] = cval[j];
            cand_pos[o] = cgid[j];
          }
        }
      }
      return;
    }
    if (C <= kCandMax) {                                  // uniform over the workgroup
#pragma unroll
      for (int e = 0; e < EPT; ++e)
        if ((flags >> e) & 1u) {
          s_cv[off] = v[e];
          s_cp[off] = p0 + e;
          ++off;
        }
      __syncthreads();
      for (int t = tid; t < (C > k ? C : k); t += 64 * nwl) {
        int64_t o;
        int pos = -1;
        float val = -INFINITY;
        int rank = t;                                       // padding slots when fewer than k exist
        int gid = -1;
        if (t < C) {
          val = s_cv[t];
          pos = s_cp[t];
          if (fin) gid = ids ? ids[b * ids_stride + pos] : pos;   // in flight while the candidate is ranked
          rank = 0;
#pragma unroll 4
          for (int q = 0; q < C; ++q) {
            const float ov = s_cv[q];
            rank += (ov > val || (ov == val && q < t)) ? 1 : 0;   // list order is position order
          }
        }
        if (rank < k) {
          if (fin) {
            o = row * k + rank;
            out_ids[o] = gid;
            if (out_vals) out_vals[o] = (LSE && val != -INFINITY) ? val - lse : val;
          } else {
            o = (row * gridDim.x + c) * k + rank;
            cand_val[o] = val;
            cand_pos[o] = pos;
          }
        }
      }
      return;
    }
  }
  // ---- general path: k rounds per wavefront, then over the wavefronts' winners
  const int wbase = cbase + wave * 64 * EPT;
  wave_select<EPT>(v, k, lane, [&](int r, float val, int pos) {
    if (lane == 0) {
      s_val[wave * k + r] = val;
      s_pos[wave * k + r] = wbase + pos;
    }
  });
  __syncthreads();
  if (wave != 0) return;
  float v2[E2];
#pragma unroll
  for (int e = 0; e < E2; ++e) {
    const int q = lane * E2 + e;
    v2[e] = (q < NW * k) ? s_val[q] : -INFINITY;
  }
  // lane r keeps the r-th winner; ids are looked up and stored by k lanes at once afterwards, so the
  // dependent id loads overlap instead of costing one round trip per rank
  float wval = -INFINITY;
  int wq = 0;
  wave_select<E2>(v2, k, lane, [&](int r, float val, int q) {
    if (lane == r) {
      wval = val;
      wq = q;
    }
  });
  if (lane < k) {
    const bool none = (wval == -INFINITY);
    const int pos = none ? -1 : s_pos[wq];
    if (fin) {
      const int64_t o = row * k + lane;
      out_ids[o] = none ? -1 : (ids ? ids[b * ids_stride + pos] : pos);
      if (out_vals) out_vals[o] = (LSE && !none) ? wval - lse : wval;
    } else {
      const int64_t o = (row * gridDim.x + c) * k + lane;
      cand_val[o] = wval;
      cand_pos[o] = pos;
    }
  }
}

template <int EPT, int NW, bool FINAL, bool LSE>
__global__ __launch_bounds__(64 * NW) void topk_select_kernel(const float* __restrict__ logits, int64_t ld,
                                                             const int32_t* __restrict__ ids, int64_t ids_stride,
                                                             const int32_t* __restrict__ n_dev, int n_fixed, int M, int k,
                                                             int32_t* __restrict__ out_ids, float* __restrict__ out_vals,
                                                             float* __restrict__ cand_val, int32_t* __restrict__ cand_pos,
                                                             float2* __restrict__ cand_ms) {
  topk_select<EPT, NW, FINAL, LSE>(logits, ld, ids, ids_stride, n_dev, n_fixed, M, k, out_ids, out_vals, cand_val, cand_pos, cand_ms);
}

// Long rows (more positions than one workgroup's registers hold): one workgroup per row walks it in pieces of 16 logits
// per thread, two pieces' loads in flight behind the one that is worked on.  The first piece gives a threshold exactly as
// above; what reaches it goes to a list in LDS, the list's k-th best becomes the threshold, and of the later pieces only
// what is strictly greater is appended (an equal value at a higher position loses the tie against k earlier ones).
// A full list is cut back to its k best.  A piece that alone overflows it (a ramp, thousands of equal values) raises the
// threshold to the exact k-th largest lane maximum: fewer than k lanes then hold anything greater (16 values each at most, they
// fit), and of the values equal to it the k first by position.
// The final order is by (value, position) explicitly, so slots are handed out by an atomic counter.
// Bound by the row's bytes; a thread's loads are consecutive 16-byte pieces across the workgroup from the row's first
// aligned element on -- the up to three elements before it and after the last whole piece are single loads -- so rows of
// any stride stream at the same rate.
constexpr int kStreamList = 2048;

template <int NW, bool LSE>
__device__ __forceinline__ void topk_stream(const float* __restrict__ logits, int64_t ld, const int32_t* __restrict__ ids, int64_t ids_stride,
                                            const int32_t* __restrict__ n_dev, int n_fixed, int M, int k, int32_t* __restrict__ out_ids,
                                            float* __restrict__ out_vals) {
  constexpr int NT = 64 * NW, QP = 4 * NT;                 // threads; 16-byte pieces per step
  __shared__ __attribute__((aligned(16))) float s_v[kStreamList + 4];
  __shared__ __attribute__((aligned(16))) int s_p[kStreamList + 4];
  __shared__ int s_r[kStreamList];
  __shared__ int s_n;
  __shared__ float s_thr[NW], s_max[NW], s_sum[NW];
  __shared__ float s_kth;
  __shared__ int s_eq[NW];
  const int m = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row = (int64_t)b * M + m;
  const float* src = logits + row * ld;
  const int head = (int)((16u - ((uint32_t)reinterpret_cast<uintptr_t>(src) & 15u)) & 15u) >> 2;   // elements before the first aligned one
  const float4* base = reinterpret_cast<const float4*>(src + head);
  const int qcap = (int)((ld - head) >> 2);                // whole pieces inside the row's stride (the launcher sends long rows only)
  float4 x[3][4];
  auto load = [&](int p, float4(&v)[4]) {                  // unconditional: past the end the last piece again, masked later
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int q = p * QP + j * NT + tid;
      v[j] = base[q < qcap ? q : qcap - 1];
    }
  };
  load(0, x[0]);
  load(1, x[1]);
  const int n = n_dev ? n_dev[b] : n_fixed;
  const int nq = n > head ? (n - head) >> 2 : 0;
  const int steps = nq > QP ? (nq + QP - 1) / QP : 1;
  // the elements outside the whole pieces: threads 0-3 before, 4-7 behind
  const int xpos = tid < 4 ? (tid < head ? tid : n) : head + 4 * nq + tid - 4;
  const bool has_x = tid < 8 && xpos < n && xpos < ld;
  const float xv = has_x ? src[xpos] : -INFINITY;
  if (tid == 0) s_n = 0;

  float T = -INFINITY;                                     // at least k elements so far are >= T (or T is -inf)
  int held = 0;                                            // list entries before the piece; both uniform over the workgroup
  float lm = has_x ? xv : -INFINITY, ls = has_x ? 1.f : 0.f;   // this thread's running maximum and sum of exp(z - maximum)

  // k-th largest over the lanes' maxima, as in topk_select_kernel; one barrier
  auto vote = [&](float ml, int valid) -> float {
    int nwe = (valid + 32) / 64;
    nwe = nwe < 1 ? 1 : (nwe > NW ? NW : nwe);
    const int rounds = (k + nwe - 1) / nwe;
    float y = ml, thr = -INFINITY;
    for (int r = 0; r < rounds; ++r) {
      thr = wave_max(y);
      const unsigned long long ball = __ballot(y == thr);
      const int L = ball ? __ffsll(ball) - 1 : 0;
      if (lane == L) y = -INFINITY;
    }
    if (lane == 0) s_thr[wave] = thr;
    __syncthreads();
    float t = s_thr[0];
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) t = fminf(t, ww < nwe ? s_thr[ww] : INFINITY);
    return t;
  };
  // every list entry's rank (value descending, position ascending) into s_r; the list is complete at the call
  auto rank_list = [&](int C) {
    if (tid < 4) {
      s_v[C + tid] = __builtin_nanf("");
      s_p[C + tid] = INT_MAX;
    }
    for (int t = tid; t < C; t += NT) s_r[t] = 0;
    __syncthreads();
    const int lg = C <= 1 ? 0 : 32 - __clz(C - 1);
    const int items = ((C + 3) >> 2) << lg;
    for (int i = tid; i < items; i += NT) {
      const int t = i & ((1 << lg) - 1), q = (i >> lg) * 4;
      if (t < C) {
        const float val = s_v[t];
        const int pos = s_p[t];
        const float4 o = *reinterpret_cast<const float4*>(&s_v[q]);
        const int4 op = *reinterpret_cast<const int4*>(&s_p[q]);
        int r = (o.x > val || (o.x == val && op.x < pos)) ? 1 : 0;
        r += (o.y > val || (o.y == val && op.y < pos)) ? 1 : 0;
        r += (o.z > val || (o.z == val && op.z < pos)) ? 1 : 0;
        r += (o.w > val || (o.w == val && op.w < pos)) ? 1 : 0;
        if (r) atomicAdd(&s_r[t], r);
      }
    }
    __syncthreads();
  };
  // The list's k best stay, in order; the k-th is the threshold from here on.  Fewer than k entries (a first piece of
  // -inf and NaN, which never enter the list) all stay and there is no threshold yet.
  auto cut_back = [&](int C) {
    const int kept = C < k ? C : k;
    rank_list(C);
    float kv[kStreamList / NT];
    int kp[kStreamList / NT], kr[kStreamList / NT];
#pragma unroll
    for (int i = 0; i < kStreamList / NT; ++i) {
      const int t = tid + i * NT;
      kr[i] = t < C ? s_r[t] : k;
      kv[i] = t < C ? s_v[t] : 0.f;
      kp[i] = t < C ? s_p[t] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kStreamList / NT; ++i)
      if (kr[i] < k) {
        s_v[kr[i]] = kv[i];
        s_p[kr[i]] = kp[i];
      }
    if (tid == 0) s_n = kept;
    __syncthreads();
    T = C < k ? -INFINITY : s_v[k - 1];
    held = kept;
  };
  auto append = [&](const float4(&v)[4], int p, float t, bool equal_too) {
    uint32_t f = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool in = p * QP + j * NT + tid < nq;
      f |= (uint32_t)(in && (v[j].x > t || (equal_too && v[j].x == t))) << (4 * j);
      f |= (uint32_t)(in && (v[j].y > t || (equal_too && v[j].y == t))) << (4 * j + 1);
      f |= (uint32_t)(in && (v[j].z > t || (equal_too && v[j].z == t))) << (4 * j + 2);
      f |= (uint32_t)(in && (v[j].w > t || (equal_too && v[j].w == t))) << (4 * j + 3);
    }
    if (f) {
      int at = atomicAdd(&s_n, __popc(f));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float e4[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((f >> (4 * j + e)) & 1u) {
            if (at < kStreamList) {
              s_v[at] = e4[e];
              s_p[at] = head + 4 * (p * QP + j * NT + tid) + e;
            }
            ++at;
          }
      }
    }
  };
  // The piece's values do not fit the list (uniform; the list holds `held` entries of earlier pieces, kStreamList / 4 at most)
  auto overflow = [&](const float4(&v)[4], int p, float ml) {
    static_assert(kStreamList - kStreamList / 4 >= NT && kStreamList - kStreamList / 4 >= 16 * kMaxK + kMaxK + 8, "room behind the held entries");
    __syncthreads();                                       // everybody knows that it overflowed
    float* lane_max = s_v + (kStreamList - NT);
    lane_max[tid] = ml;
    if (tid == 0) s_n = held;
    __syncthreads();
    int r = 0;
    for (int q = 0; q < NT; q += 4) {
      const float4 o = *reinterpret_cast<const float4*>(&lane_max[q]);
      r += (o.x > ml || (o.x == ml && q < tid)) + (o.y > ml || (o.y == ml && q + 1 < tid)) + (o.z > ml || (o.z == ml && q + 2 < tid)) +
           (o.w > ml || (o.w == ml && q + 3 < tid));
    }
    if (r == k - 1) s_kth = ml;                            // ranks are distinct and k <= 64 <= NT: one thread
    __syncthreads();
    const float t = s_kth;
    const bool raised = t > T || p == 0;                   // else: nothing equal to T is wanted, and fewer than k lanes hold more
    if (raised) T = t;
    append(v, p, T, false);
    if (raised) {
      int taken = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {                        // position order: j, then thread, then element
        const float e4[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
        const bool in = p * QP + j * NT + tid < nq;
        int mine = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) mine += (in && e4[e] == T) ? 1 : 0;
        int incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int u = __shfl_up(incl, o);
          incl += lane >= o ? u : 0;
        }
        if (lane == 63) s_eq[wave] = incl;
        __syncthreads();
        int off = incl - mine, tot = 0;
        for (int ww = 0; ww < NW; ++ww) {
          off += ww < wave ? s_eq[ww] : 0;
          tot += s_eq[ww];
        }
        off += taken;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (in && e4[e] == T) {
            if (off < k) {
              const int at = atomicAdd(&s_n, 1);
              s_v[at] = e4[e];
              s_p[at] = head + 4 * (p * QP + j * NT + tid) + e;
            }
            ++off;
          }
        taken += tot;
        __syncthreads();
      }
    }
  };
  auto process = [&](float4(&v)[4], int p) {
    float ml = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool in = p * QP + j * NT + tid < nq;
      v[j].x = in ? v[j].x : -INFINITY;
      v[j].y = in ? v[j].y : -INFINITY;
      v[j].z = in ? v[j].z : -INFINITY;
      v[j].w = in ? v[j].w : -INFINITY;
      ml = fmaxf(ml, fmaxf(fmaxf(v[j].x, v[j].y), fmaxf(v[j].z, v[j].w)));
    }
    if (LSE) {
      const float nm = fmaxf(lm, ml);
      const float ref = nm == -INFINITY ? 0.f : nm;
      float se = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) se += (__expf(v[j].x - ref) + __expf(v[j].y - ref)) + (__expf(v[j].z - ref) + __expf(v[j].w - ref));
      ls = ls * expf(lm - ref) + se;                       // lm == -inf: the factor is 0
      lm = nm;
    }
    const int valid = nq - p * QP < NT ? nq - p * QP : NT;
    if (p == 0) T = vote(ml, valid);                       // its barrier also publishes s_n = 0
    append(v, p, T, p == 0 && T != -INFINITY);             // -inf is no candidate: it is what an empty slot holds
    __syncthreads();
    int C = s_n;
    if (C > kStreamList - 8) {                             // uniform; eight entries are kept for the elements outside the pieces
      overflow(v, p, ml);
      __syncthreads();
      C = s_n;
    }
    if (p + 1 < steps && (p == 0 || C > kStreamList / 4)) {
      cut_back(C);
    } else {
      __syncthreads();                                     // s_n has been read by all before the next piece adds to it
      held = C;
    }
  };
  for (int p = 0; p < steps; p += 3) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      load(p + j + 2, x[(j + 2) % 3]);
      if (p + j < steps) process(x[j], p + j);
    }
  }

  float lse = 0.f;
  if (LSE) {                                               // lanes, then wavefronts, in a fixed order
    const float wm = wave_max(lm);
    const float ws = wave_add(ls * expf(lm - (wm == -INFINITY ? 0.f : wm)));
    if (lane == 0) {
      s_max[wave] = wm;
      s_sum[wave] = ws;
    }
    __syncthreads();
    const float pm = lane < NW ? s_max[lane] : -INFINITY;
    float zmax = wave_max(pm);
    zmax = zmax == -INFINITY ? 0.f : zmax;
    lse = zmax + logf(wave_add(lane < NW ? s_sum[lane] * expf(pm - zmax) : 0.f));
  }
  auto write = [&](int r, int pos, float val, int gid) {
    out_ids[row * k + r] = gid;
    if (out_vals) out_vals[row * k + r] = (LSE && val != -INFINITY) ? val - lse : val;
  };
  if (has_x && xv > -INFINITY) {                           // neither a NaN, which has no rank, nor -inf; a superset of the winners is listed: the rank decides
    const int at = atomicAdd(&s_n, 1);
    s_v[at] = xv;
    s_p[at] = xpos;
  }
  __syncthreads();
  const int C = s_n;
  {
    int gid[kStreamList / NT];                             // requested before the ranking, used behind it
#pragma unroll
    for (int i = 0; i < kStreamList / NT; ++i) {
      const int t = tid + i * NT;
      gid[i] = t < C ? s_p[t] : 0;
      if (ids && t < C) gid[i] = ids[b * ids_stride + gid[i]];
    }
    __syncthreads();
    rank_list(C);
#pragma unroll
    for (int i = 0; i < kStreamList / NT; ++i) {
      const int t = tid + i * NT;
      if (t < C && s_r[t] < k) write(s_r[t], s_p[t], s_v[t], gid[i]);
    }
  }
  if (tid >= C && tid < k) {                            // padding slots when fewer than k exist
    out_ids[row * k + tid] = -1;
    if (out_vals) out_vals[row * k + tid] = -INFINITY;
  }
}

template <int NW>
__global__ __launch_bounds__(64 * NW) void topk_stream_kernel(const float* __restrict__ logits, int64_t ld, int n, int M, int k,
                                                              int32_t* __restrict__ out_ids, float* __restrict__ out_vals) {
  topk_stream<NW, false>(logits, ld, nullptr, 0, nullptr, n, M, k, out_ids, out_vals);
}

// Lists whose capacity is beyond one workgroup's registers but whose live row count mostly is not: one launch that selects
// either way, by the count on the device.  (Sixteen wavefronts with log-probabilities keep 28 bytes a lane in scratch memory, all on the walk; a short list does not
// show it: 8 rows of 3000 ids 4.5 us, with log-probabilities 5.0; the chunk kernels' 5.8 and 6.4.)
template <int NW, bool LSE>
__global__ __launch_bounds__(64 * NW) void topk_list_kernel(const float* __restrict__ logits, int64_t ld, const int32_t* __restrict__ ids,
                                                            int64_t ids_stride, const int32_t* __restrict__ n_dev, int n_fixed, int M, int k,
                                                            int32_t* __restrict__ out_ids, float* __restrict__ out_vals) {
  if ((n_dev ? n_dev[blockIdx.z] : n_fixed) <= NW * 1024)
    topk_select<16, NW, true, LSE>(logits, ld, ids, ids_stride, n_dev, n_fixed, M, k, out_ids, out_vals, nullptr, nullptr, nullptr);
  else
    topk_stream<NW, LSE>(logits, ld, ids, ids_stride, n_dev, n_fixed, M, k, out_ids, out_vals);
}

// Merge the per-chunk winners of one row (nchunks*k <= 1024 candidates, in position order): one candidate per thread, its rank
// among all of them as (candidate, group of four) work items over the workgroup.  (17 rows of 128256, k = 40,
// selection and merge: 24.9 -> 19.7 us against rounds of one wavefront; k = 10 11.9 -> 9.6; 8 rows of 32000, k = 40 22.9 -> 9.1; 256
// threads instead of 1024: k = 40 39 us.)
template <bool LIST, bool LSE>   // LIST: not dense rows, whose positions are the ids and whose length is known to need the chunks
__global__ __launch_bounds__(1024) void topk_merge_kernel(const float* __restrict__ cand_val, const int32_t* __restrict__ cand_pos,
                                                          const float2* __restrict__ cand_ms, int nchunks,
                                                          const int32_t* __restrict__ ids, int64_t ids_stride, int M, int k,
                                                          int32_t* __restrict__ out_ids, float* __restrict__ out_vals,
                                                          const int32_t* __restrict__ n_dev) {
  __shared__ __attribute__((aligned(16))) float s_v[1024 + 4];
  __shared__ int s_r[1024];
  const int tid = threadIdx.x, lane = tid & 63;
  const int m = blockIdx.y, b = blockIdx.z;
  if (LIST && n_dev[b] <= kTopkChunk) return;               // the first chunk's workgroup has written the result
  const int64_t row = (int64_t)b * M + m;
  const int total = nchunks * k;
  float val = -INFINITY;
  int pos = -1;
  if (tid < total) {
    val = cand_val[row * total + tid];
    pos = cand_pos[row * total + tid];
    s_v[tid] = val;
    s_r[tid] = 0;
  }
  if (tid < 4) s_v[total + tid] = __builtin_nanf("");       // pads the last group of four; compares false with everything
  const int gid = LIST && val != -INFINITY ? ids[b * ids_stride + pos] : pos;   // requested before the ranking, used behind it
  float lse = 0.f;
  if (LSE) {                                              // chunk (max, sum) pairs -> one log sum exp; at most 16 chunks
    const float2 ms = lane < nchunks ? cand_ms[row * nchunks + lane] : make_float2(0.f, 0.f);
    float zmax = wave_max(ms.y > 0.f ? ms.x : -INFINITY);
    zmax = zmax == -INFINITY ? 0.f : zmax;
    lse = zmax + logf(wave_add(ms.y > 0.f ? ms.y * expf(ms.x - zmax) : 0.f));
  }
  __syncthreads();
  const int lg = total <= 1 ? 0 : 32 - __clz(total - 1);
  const int items = ((total + 3) >> 2) << lg;
  for (int w = tid; w < items; w += 1024) {
    const int t = w & ((1 << lg) - 1), q = (w >> lg) * 4;
    if (t < total) {
      const float x = s_v[t];
      const float4 o = *reinterpret_cast<const float4*>(&s_v[q]);
      int r = (o.x > x || (o.x == x && q < t)) ? 1 : 0;             // list order is position order
      r += (o.y > x || (o.y == x && q + 1 < t)) ? 1 : 0;
      r += (o.z > x || (o.z == x && q + 2 < t)) ? 1 : 0;
      r += (o.w > x || (o.w == x && q + 3 < t)) ? 1 : 0;
      if (r) atomicAdd(&s_r[t], r);
    }
  }
  __syncthreads();
  if (tid < total && s_r[tid] < k) {
    const bool none = val == -INFINITY;                     // fewer than k exist
    const int64_t o = row * k + s_r[tid];
    out_ids[o] = none ? -1 : gid;
    if (out_vals) out_vals[o] = (LSE && !none) ? val - lse : val;
  }
}

static int chunks_for(int32_t cap) { return (cap + kTopkChunk - 1) / kTopkChunk; }

// What the chunks of these rows need.  It is asked for at every size, also where one workgroup per row or per list runs and leaves it
// unused, so that what a caller has to hold and what is refused does not change with the choice of the kernel.
int64_t topk_workspace_bytes(int32_t cap, int32_t rows, int32_t k) {
  if (cap <= kTopkChunk) return 0;
  return (int64_t)rows * chunks_for(cap) * (k * 8 + 8);   // (value, position) per winner + (max, sum) per chunk
}

template <bool LSE>
static hipError_t launch_topk_t(const float* logits, int64_t ld, const int32_t* ids, int64_t ids_stride, const int32_t* n_dev,
                                int32_t n_fixed, int32_t cap, int64_t expected, int32_t batch, int32_t M, int32_t k, int32_t* out_ids,
                                float* out_vals, char* ws, int64_t ws_bytes, hipStream_t s) {
  const dim3 rows(1, M, batch);
  if (LSE && !n_dev) return hipErrorInvalidValue;           // log-probabilities are taken over lists only
  if (cap <= 4096) {
    topk_select_kernel<16, 4, true, LSE><<<rows, 256, 0, s>>>(logits, ld, ids, ids_stride, n_dev, n_fixed, M, k, out_ids,
                                                            out_vals, nullptr, nullptr, nullptr);
    return hipGetLastError();
  }
  if (cap <= 8192) {   // eight wavefronts beat sixteen (c3: 6.2 -> 5.0 us, c4: 8.2 -> 5.8 us) and four with 32 logits per lane (5.5, 6.1)
    topk_select_kernel<16, 8, true, LSE><<<rows, 512, 0, s>>>(logits, ld, ids, ids_stride, n_dev, n_fixed, M, k, out_ids,
                                                            out_vals, nullptr, nullptr, nullptr);
    return hipGetLastError();
  }
  if (cap <= kTopkChunk) {
    topk_select_kernel<16, 16, true, LSE><<<rows, 1024, 0, s>>>(logits, ld, ids, ids_stride, n_dev, n_fixed, M, k, out_ids,
                                                              out_vals, nullptr, nullptr, nullptr);
    return hipGetLastError();
  }
  const int nch = chunks_for(cap);
  const int64_t need = topk_workspace_bytes(cap, batch * M, k);
  if (nch * k > 1024 || ws == nullptr || ws_bytes < need) return hipErrorInvalidValue;
  const int64_t nrows = (int64_t)batch * M;
  if (!topk_chunks(n_dev != nullptr, nrows, k, expected)) {
    // Eight wavefronts instead of sixteen from 512 rows on (2048 rows of 32000, k = 5: 52 against 77 us; 500 rows of 50001, k = 40: 45 against 42); lists that fit
    // those registers -- 8192 ids -- are selected as short ones there too (512 rows, 3000 of 32768 ids: k = 10 5.6 against 14.3 us in
    // steps and 15.6 in chunks, k = 40 8.6 / 18.2 / 18.2; 2048 rows, k = 40 24 / 46 / 48; 32000 ids 20.0 / 19.5 / 31.6).
    if (n_dev) {
      if (nrows >= 512) topk_list_kernel<8, LSE><<<rows, 512, 0, s>>>(logits, ld, ids, ids_stride, n_dev, n_fixed, M, k, out_ids, out_vals);
      else topk_list_kernel<16, LSE><<<rows, 1024, 0, s>>>(logits, ld, ids, ids_stride, n_dev, n_fixed, M, k, out_ids, out_vals);
    } else if constexpr (!LSE) {
      if (nrows >= 512) topk_stream_kernel<8><<<rows, 512, 0, s>>>(logits, ld, n_fixed, M, k, out_ids, out_vals);
      else topk_stream_kernel<16><<<rows, 1024, 0, s>>>(logits, ld, n_fixed, M, k, out_ids, out_vals);
    }
    return hipGetLastError();
  }
  const int64_t slots = (int64_t)batch * M * nch * k;
  float* cv = reinterpret_cast<float*>(ws);
  int32_t* cp = reinterpret_cast<int32_t*>(ws + slots * 4);
  float2* ms = reinterpret_cast<float2*>(ws + slots * 8);
  topk_select_kernel<16, 16, false, LSE><<<dim3(nch, M, batch), 1024, 0, s>>>(logits, ld, ids, ids_stride, n_dev, n_fixed, M, k, out_ids,
                                                                            out_vals, cv, cp, ms);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (n_dev) topk_merge_kernel<true, LSE><<<rows, 1024, 0, s>>>(cv, cp, ms, nch, ids, ids_stride, M, k, out_ids, out_vals, n_dev);
  else if constexpr (!LSE) topk_merge_kernel<false, false><<<rows, 1024, 0, s>>>(cv, cp, ms, nch, ids, ids_stride, M, k, out_ids, out_vals, n_dev);
  return hipGetLastError();
}

hipError_t launch_topk(const float* logits, int64_t ld, const int32_t* ids, int64_t ids_stride, const int32_t* n_dev,
                       int32_t n_fixed, int32_t cap, int64_t expected, int32_t batch, int32_t M, int32_t k, int32_t* out_ids,
                       float* out_vals, bool logprob, char* ws, int64_t ws_bytes, hipStream_t s) {
  return logprob ? launch_topk_t<true>(logits, ld, ids, ids_stride, n_dev, n_fixed, cap, expected, batch, M, k, out_ids, out_vals, ws,
                                       ws_bytes, s)
                 : launch_topk_t<false>(logits, ld, ids, ids_stride, n_dev, n_fixed, cap, expected, batch, M, k, out_ids, out_vals, ws,
                                        ws_bytes, s);
}

}  // namespace nanospec
