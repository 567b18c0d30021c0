// Several sequences in one batch (multi-sequence serving; Sec. 4.6 notes that the per-sequence cost of the method
// adds up over the batch): sequences that draw from one token distribution hold many of the same ids, and the
// per-sequence head fetches such a row once per sequence that holds it.  Here the active sets are split:
//   * an id held by at least min_share sequences is a *shared* row -- listed once (ascending, at most shared_cap
//     of them), fetched once and multiplied with the hidden rows of all sequences; a sequence that does not hold
//     it simply has no column for it;
//   * everything else stays on a per-sequence list and goes through the per-sequence head as before.
// The per-sequence head's launch order finds most shared rows in cache, so that the split is the faster way only where the lists overlap enough (union_split_pairs
// in choose.h); elsewhere the head is given every list whole.
// Every (sequence, active id) pair is covered by exactly one of the two parts and its logit lands in the column
// the id has in that sequence's ascending active list, so the logits have the layout of nanospec_sparse_head and
// the selection applies unchanged.
#include "common.h"

namespace nanospec {

constexpr int kListThreads = 1024;

// acc += x, bit planes of 32 counts side by side (plane k holds bit k of each)
template <int N, int NX>
__device__ __forceinline__ void planes_add(uint32_t (&acc)[N], const uint32_t (&x)[NX]) {
  uint32_t carry = 0u;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const uint32_t y = k < NX ? x[k] : 0u, half = acc[k] ^ y, out = (acc[k] & y) | (half & carry);
    acc[k] = half ^ carry;
    carry = out;
  }
}

// Sixteen bitmap words (window bitmap | T bitmap) per workgroup, a row of 16 lanes each of them for one sequence: 64 bytes in one piece.  A thread adds its word of
// sequences g, g + 16, ... into bit planes (32 counts at once, P planes), sixteen such sums meet in LDS, and the ids whose count reaches min_share are a borrow chain over the planes.
// What bounds it is the round trip of its loads.  A wavefront per word with a sequence to each lane and 32 ballots, as before, took a cache line per lane and load, and its 160 scalar
// instructions a wavefront share one scalar unit.  With the lists behind it: 64 sequences of 2300, V = 128256 9.0 -> 7.65 us, 16 of 600, V = 32000 6.9 -> 6.0, 130 of 8000, V = 152064
// 21.3 -> 16.0, 256 of 2000, V = 128256 14.2 -> 11.0.  The two halves of a cache line on one die: the same.
// u.parts, where kept: per workgroup the pairs of a sequence and an active id, and those of ids that qualify as shared.
constexpr int kCountThreads = 256;
template <int P>
__global__ __launch_bounds__(kCountThreads) void union_count_kernel(VocabPtrs p, UnionPtrs u, int batch) {
  constexpr int G = kCountThreads / 16, N = P + 4;                       // at most 2^(P - 1) words a thread, 16 threads a word
  static_assert(G == 16, "four groups to a lane of the first wavefront, four lanes to a word");
  __shared__ uint32_t s_plane[P][kCountThreads];
  const int tid = threadIdx.x, lane = tid & 63, g = tid >> 4, w = blockIdx.x * 16 + (tid & 15);
  const bool in = w < p.nwords;
  uint32_t pl[P];
#pragma unroll
  for (int k = 0; k < P; ++k) pl[k] = 0u;
  for (int s0 = 0; s0 < batch; s0 += 4 * G) {
    uint32_t v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int s = s0 + j * G + g;
      const size_t at = (size_t)(s < batch ? s : 0) * p.nwords + (in ? w : 0);
      v[j] = p.wbit[at] | p.tbit[at];
      v[j] = in && s < batch ? v[j] : 0u;
    }
    const uint32_t h1 = v[0] ^ v[1], one = h1 ^ v[2], c1 = (v[0] & v[1]) | (h1 & v[2]), c2 = one & v[3];
    planes_add(pl, {one ^ v[3], c1 ^ c2, c1 & c2});
  }
#pragma unroll
  for (int k = 0; k < P; ++k) s_plane[k][tid] = pl[k];
  __syncthreads();
  if (tid >= 64) return;
  uint32_t sum[N];
#pragma unroll
  for (int k = 0; k < N; ++k) sum[k] = 0u;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t x[P];
#pragma unroll
    for (int k = 0; k < P; ++k) x[k] = s_plane[k][j * 64 + lane];
    planes_add(sum, x);
  }
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) {
    uint32_t x[N];
#pragma unroll
    for (int k = 0; k < N; ++k) x[k] = __shfl_xor(sum[k], o);
    planes_add(sum, x);
  }
  uint32_t less = 0u;                                                    // bit = that count - min_share borrows
#pragma unroll
  for (int k = 0; k < N; ++k) less = (u.min_share >> k) & 1 ? less | ~sum[k] : less & ~sum[k];
  const uint32_t pop = u.min_share >> N ? 0u : ~less;
  if (lane < 16 && in) u.shared_bits[w] = pop;
  if (u.parts) {
    int pairs = 0, cover = 0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      pairs += __popc(sum[k]) << k;
      cover += __popc(sum[k] & pop) << k;
    }
    pairs = row_sum(pairs);
    cover = row_sum(cover);
    if (lane == 0) u.parts[blockIdx.x] = make_int2(pairs, cover);
  }
}

constexpr int kListsLds = 150 * 1024;

// Per sequence, N consecutive bitmap words per thread: everything follows from the bitmaps, fetched together in one round trip.  A shared id's rank is the
// count of shared bits before it (each workgroup writes the list of its share of the words), its column in this sequence the count of active bits before it; an active bit that is not
// shared -- or whose rank finds no room on the list -- goes to the sequence's own list, at the count of such bits before it.  Three DPP scans.
// The list is then walked: its ids, coalesced, each with one look-up in an LDS table of its bitmap word -- written from the bits themselves, a thread's are as many as the list is long in its part of the ids,
// all one after the other, where ids cluster a few threads write the whole list, and nothing is coalesced.  Figures with the counts; the bits / walked, one workgroup a sequence:
// 64 lists of 2300, V = 128256 10.2 / 9.9 us, of 20000 44.6 / 20.8, 130 of 8000, V = 152064 32.3 / 21.7, 24 of 5000, V = 50000 15.4 / 10.0; with the workgroups below 64 of 300 7.1 / 6.5, 16 of 300, V = 32000 5.9 / 5.6.
// A workgroup's sixteen wavefronts share four SIMDs, so up to four workgroups (gridDim.y, as many as fill the chip) write a sequence's lists, each for `per` threads' words and from its own scans of them all:
// 64 lists of 2300 9.9 -> 9.0 us, of 20000 20.8 -> 15.3, 8 of 3000 8.8 -> 7.7, 40 of 4000, V = 262400 17.8 -> 15.5 (eight: 0.1 us less for 8 and 24 sequences; two: 0.3 more for 64).
// What the head works from (u.head_*, kept where union_feeds says so): the split, or nothing shared and every list whole, by how many pairs the listed ids cover in
// all sequences together (to the count's sixteen words); every workgroup comes to the same answer.
template <int N>
__global__ __launch_bounds__(kListThreads) void union_lists_kernel(VocabPtrs p, UnionPtrs u, int batch, int groups, int per) {
  constexpr int NW = kListThreads / 64;
  static_assert(NW == 16, "a row of lanes holds one total per wavefront");
  extern __shared__ __attribute__((aligned(16))) uint4 tab[];   // per word of this workgroup: shared bits, active shared bits, rank of the first shared bit, active shared bits before
  __shared__ int s_shared[NW], s_active[NW], s_rest[NW], s_pairs[NW], s_cover[NW], s_rank[2], s_pos[2], s_cut;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, b = blockIdx.x, w0 = tid * N;
  const int first = blockIdx.y * per, final = blockIdx.y == gridDim.y - 1;
  const bool mine = tid >= first && tid < first + per;
  const uint32_t* gw = p.wbit + (size_t)b * p.nwords;
  const uint32_t* gt = p.tbit + (size_t)b * p.nwords;
  int32_t* mypos = u.shared_pos + (size_t)b * u.shared_cap;
  const int n = p.n[b];
  uint32_t sh[N], ac[N];
  if constexpr (N == 1) {
    sh[0] = w0 < p.nwords ? u.shared_bits[w0] : 0u;
    ac[0] = w0 < p.nwords ? gw[w0] | gt[w0] : 0u;
  } else if constexpr (N == 2) {
    uint2 x = make_uint2(0, 0), y = x, z = x;
    if (w0 < p.nwords) {                                                 // nwords is a multiple of 4
      x = *reinterpret_cast<const uint2*>(u.shared_bits + w0);
      y = *reinterpret_cast<const uint2*>(gw + w0);
      z = *reinterpret_cast<const uint2*>(gt + w0);
    }
    sh[0] = x.x; sh[1] = x.y;
    ac[0] = y.x | z.x; ac[1] = y.y | z.y;
  } else {
#pragma unroll
    for (int c = 0; c < N; c += 4) {
      uint4 x = make_uint4(0, 0, 0, 0), y = x, z = x;
      if (w0 + c < p.nwords) {
        x = *reinterpret_cast<const uint4*>(u.shared_bits + w0 + c);
        y = *reinterpret_cast<const uint4*>(gw + w0 + c);
        z = *reinterpret_cast<const uint4*>(gt + w0 + c);
      }
      sh[c] = x.x; sh[c + 1] = x.y; sh[c + 2] = x.z; sh[c + 3] = x.w;
      ac[c] = y.x | z.x; ac[c + 1] = y.y | z.y; ac[c + 2] = y.z | z.z; ac[c + 3] = y.w | z.w;
    }
  }
  int2 sums = make_int2(0, 0);
  if (u.parts && tid < (p.nwords + 15) / 16) sums = u.parts[tid];        // at most 1024 of them: a state has fewer than 16384 words
  int ns = 0, na = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    ns += __popc(sh[i]);
    na += __popc(ac[i]);
  }
  const int si = wave_incl_scan(ns), ai = wave_incl_scan(na);
  if (lane == 63) {
    s_shared[wave] = si;
    s_active[wave] = ai;
  }
  if (u.parts) {
    const int pi = wave_incl_scan(sums.x);
    if (lane == 63) s_pairs[wave] = pi;
  }
  __syncthreads();
  const int ts = s_shared[lane & 15], ta = s_active[lane & 15];
  int r = row_sum((lane & 15) < wave ? ts : 0) + si - ns;                // rank of this thread's first shared bit
  int pos = row_sum((lane & 15) < wave ? ta : 0) + ai - na;              // column of its first active bit
  const int all = row_sum(ts), listed = all < u.shared_cap ? all : u.shared_cap;
  if (tid == first) {
    s_rank[0] = r < listed ? r : listed;
    s_pos[0] = pos;
  }
  if (tid == (final ? first : first + per - 1)) {
    s_rank[1] = final ? u.shared_cap : r + ns < listed ? r + ns : listed;
    s_pos[1] = final ? n : pos + na;
  }
  // the first of the count's workgroups whose ids do not all find room on the list
  if (all <= u.shared_cap ? tid == 0 : r <= u.shared_cap && r + ns > u.shared_cap) s_cut = all <= u.shared_cap ? kListThreads : w0 / 16;
  if (r + ns > u.shared_cap) {                                           // bits without room on the list are not shared
    int room = u.shared_cap - r;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      uint32_t keep = 0u;
      for (uint32_t x = sh[i]; x && room > 0; x &= x - 1u, --room) keep |= x & (0u - x);
      sh[i] = keep;
    }
  }
  int nr = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) nr += __popc(ac[i] & ~sh[i]);
  const int ri = wave_incl_scan(nr);
  if (lane == 63) s_rest[wave] = ri;
  __syncthreads();
  if (u.parts) {
    const int ci = wave_incl_scan(tid < s_cut ? sums.y : 0);
    if (lane == 63) s_cover[wave] = ci;
  }
  const int tr = s_rest[lane & 15], nrest = row_sum(tr);
  int q = row_sum((lane & 15) < wave ? tr : 0) + ri - nr;
  int32_t* rid = u.rest_ids + (size_t)b * p.cap;
  int32_t* rpos = u.rest_pos + (size_t)b * p.cap;
  int32_t* hid = u.parts ? u.head_ids + (size_t)b * p.cap : nullptr;
  int32_t* hpos = u.parts ? u.head_pos + (size_t)b * p.cap : nullptr;
  for (int i = s_rank[0] + tid; i < s_rank[1]; i += kListThreads) mypos[i] = -1;   // shared ids the sequence lacks, and room that none takes; the barrier below is between these and the columns
  if (mine && (tid * batch) >> 10 == b) {                                // this workgroup's share of the list of shared ids
    int at = r;
#pragma unroll
    for (int i = 0; i < N; ++i)
      for (uint32_t x = sh[i]; x; x &= x - 1u) u.shared_ids[at++] = (w0 + i) * 32 + __ffs(x) - 1;
  }
  if (mine) {
    int rank = r, before = pos - q;                                      // active shared bits before this thread's words
#pragma unroll
    for (int i = 0; i < N; ++i) {
      tab[(tid - first) * N + i] = make_uint4(sh[i], ac[i] & sh[i], (uint32_t)rank, (uint32_t)before);
      rank += __popc(sh[i]);
      before += __popc(ac[i] & sh[i]);
    }
  }
  __syncthreads();
  bool split = false;
  if (u.parts) {
    const int pairs = row_sum(s_pairs[lane & 15]);
    split = union_split_pairs(pairs, pairs - row_sum(s_cover[lane & 15]));
  }
  const int32_t* ids = p.ids + (size_t)b * p.cap;
  for (int j = s_pos[0] + tid; j < s_pos[1]; j += kListThreads) {
    const int id = ids[j];
    const uint4 t = tab[(id >> 5) - first * N];
    const uint32_t below = (1u << (id & 31)) - 1u;
    if ((t.x >> (id & 31)) & 1u) {
      mypos[t.z + __popc(t.x & below)] = j;
    } else {
      const int at = j - (int)t.w - __popc(t.y & below);
      rid[at] = id;
      rpos[at] = j;
      if (hid && split) {
        hid[at] = id;
        hpos[at] = j;
      }
    }
    if (hid && !split) {
      hid[j] = id;
      hpos[j] = j;
    }
  }
  if (b == 0 && final)
    for (int g = tid; g < groups; g += kListThreads) {
      u.shared_n[g] = listed;
      if (hid) u.head_shared_n[g] = split ? listed : 0;
    }
  if (final && tid == 0) {
    u.rest_n[b] = nrest;
    if (hid) u.head_n[b] = split ? nrest : n;
  }
}

__global__ __launch_bounds__(256) void union_reset_kernel(UnionPtrs u, int batch, int cap, int groups) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, stride = (int64_t)gridDim.x * 256;
  for (int64_t x = i; x < (int64_t)batch * cap; x += stride) {
    u.rest_ids[x] = 0;
    u.rest_pos[x] = -1;
  }
  for (int64_t x = i; x < (int64_t)batch * u.shared_cap; x += stride) u.shared_pos[x] = -1;
  for (int64_t x = i; x < u.shared_cap; x += stride) u.shared_ids[x] = 0;
  for (int64_t x = i; x < batch; x += stride) u.rest_n[x] = 0;
  for (int64_t x = i; x < groups; x += stride) u.shared_n[x] = 0;
  if (!u.parts) return;
  for (int64_t x = i; x < (int64_t)batch * cap; x += stride) {
    u.head_ids[x] = 0;
    u.head_pos[x] = -1;
  }
  for (int64_t x = i; x < batch; x += stride) u.head_n[x] = 0;
  for (int64_t x = i; x < groups; x += stride) u.head_shared_n[x] = 0;
}

hipError_t union_configure_device() {
  const void* fns[] = {reinterpret_cast<const void*>(union_lists_kernel<1>), reinterpret_cast<const void*>(union_lists_kernel<2>), reinterpret_cast<const void*>(union_lists_kernel<4>),
                       reinterpret_cast<const void*>(union_lists_kernel<8>), reinterpret_cast<const void*>(union_lists_kernel<16>)};
  for (const void* f : fns) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kListsLds);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_union_reset(const nanospec_state* st, hipStream_t s) {
  union_reset_kernel<<<256, 256, 0, s>>>(st->un, st->batch, st->vp.cap, st->un_groups);
  return hipGetLastError();
}

hipError_t launch_union_build(const nanospec_state* st, hipStream_t s) {
  const int nw = st->vp.nwords;
  static_assert(NANOSPEC_MAX_BATCH <= 256, "sixteen words a thread");
  if (st->batch <= 64) union_count_kernel<3><<<(nw + 15) / 16, kCountThreads, 0, s>>>(st->vp, st->un, st->batch);
  else union_count_kernel<5><<<(nw + 15) / 16, kCountThreads, 0, s>>>(st->vp, st->un, st->batch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int N = nw <= kListThreads ? 1 : nw <= 2 * kListThreads ? 2 : nw <= 4 * kListThreads ? 4 : nw <= 8 * kListThreads ? 8 : 16;
  const int parts = st->batch <= 64 ? 4 : st->batch <= 128 || 16ll * nw > kListsLds ? 2 : 1;              // as many workgroups as compute units, and tables that fit LDS
  const int per = ((nw + N - 1) / N + parts - 1) / parts, lds = per * N * 16;
  const dim3 grid(st->batch, parts);
  if (nw > 16 * kListThreads || lds > kListsLds) return hipErrorInvalidValue;   // more ids than a state takes: its bitmaps fill LDS three times over
  if (N == 1) union_lists_kernel<1><<<grid, kListThreads, lds, s>>>(st->vp, st->un, st->batch, st->un_groups, per);
  else if (N == 2) union_lists_kernel<2><<<grid, kListThreads, lds, s>>>(st->vp, st->un, st->batch, st->un_groups, per);
  else if (N == 4) union_lists_kernel<4><<<grid, kListThreads, lds, s>>>(st->vp, st->un, st->batch, st->un_groups, per);
  else if (N == 8) union_lists_kernel<8><<<grid, kListThreads, lds, s>>>(st->vp, st->un, st->batch, st->un_groups, per);
  else union_lists_kernel<16><<<grid, kListThreads, lds, s>>>(st->vp, st->un, st->batch, st->un_groups, per);
  return hipGetLastError();
}

}  // namespace nanospec
