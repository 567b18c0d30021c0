// Several sequences in one batch (multi-sequence serving; Sec. 4.6 notes that the per-sequence cost of the method
// adds up over the batch): sequences that draw from one token distribution hold many of the same ids, and the
// per-sequence head fetches such a row once per sequence that holds it.  Here the active sets are split:
//   * an id held by at least min_share sequences is a *shared* row -- listed once (ascending, at most shared_cap
//     of them), fetched once and multiplied with the hidden rows of all sequences; a sequence that does not hold
//     it simply has no column for it;
//   * everything else stays on a per-sequence list and goes through the per-sequence head as before.
// Every (sequence, active id) pair is covered by exactly one of the two parts and its logit lands in the column
// the id has in that sequence's ascending active list, so the logits have the layout of nanospec_sparse_head and
// the selection applies unchanged.
#include "common.h"

namespace nanospec {

constexpr int kListThreads = 1024;

// One wavefront per bitmap word: lane q looks at sequence q's word (window bitmap | T bitmap); 32 ballots count,
// for every bit, the sequences that hold the id.  (Four words to a wavefront, sixteen bytes a lane: 1.9 us slower, a chain of 128 ballots.)  FEED: u.parts gets, per workgroup, the
// pairs of a sequence and an active id, and those of ids that qualify as shared.
template <bool FEED>
__global__ __launch_bounds__(1024) void union_count_kernel(VocabPtrs p, UnionPtrs u, int batch) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int w = blockIdx.x * 16 + wave;
  if (!FEED && w >= p.nwords) return;
  constexpr int NB = (NANOSPEC_MAX_BATCH + 63) / 64;
  uint32_t word[NB];
  int cnt[32];
#pragma unroll
  for (int i = 0; i < 32; ++i) cnt[i] = 0;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    word[k] = 0u;
    if (k * 64 >= batch) continue;
    const int b = k * 64 + lane;
    if (b < batch && (!FEED || w < p.nwords)) word[k] = p.wbit[(size_t)b * p.nwords + w] | p.tbit[(size_t)b * p.nwords + w];
#pragma unroll
    for (int i = 0; i < 32; ++i) cnt[i] += __popcll(__ballot((word[k] >> i) & 1u));
  }
  uint32_t pop = 0u;
#pragma unroll
  for (int i = 0; i < 32; ++i) pop |= (cnt[i] >= u.min_share ? 1u : 0u) << i;
  if (lane == 0 && (!FEED || w < p.nwords)) u.shared_bits[w] = pop;
  if constexpr (FEED) {
    __shared__ int s_sum[16];
    int both = 0;                                                        // at most 8192 pairs to a word: two sums in one register
#pragma unroll
    for (int k = 0; k < NB; ++k) both += __popc(word[k]) << 16 | __popc(word[k] & pop);
    both = wave_incl_scan(both);
    if (lane == 63) s_sum[wave] = both;
    __syncthreads();
    if (wave == 0) {
      const int x = s_sum[lane & 15], a = row_sum(x >> 16), c = row_sum(x & 0xffff);
      if (lane == 0) u.parts[blockIdx.x] = make_int2(a, c);
    }
  }
}

// Lists longer than this are walked, shorter ones written from the bits (see union_lists_kernel).
constexpr int kWalkFrom = 1024;
constexpr int kListsLds = 150 * 1024;

// One workgroup per sequence, N consecutive bitmap words per thread: everything follows from the bitmaps, fetched together in one round trip.  A shared id's rank is the
// count of shared bits before it (each workgroup writes the list of its share of the words), its column in this sequence the count of active bits before it; an active bit that is not
// shared -- or whose rank finds no room on the list -- goes to the sequence's own list, at the count of such bits before it.  Three DPP scans, two barriers.
// Long lists are walked instead: their ids, coalesced, each with one look-up in an LDS table of its bitmap word -- a thread's bits are as many as the list is long in its part of the ids, all
// one after the other, where ids cluster a few threads write the whole list, and nothing is coalesced.  Against the walk with two look-ups and a rank per id that came before the bits / the bits alone, with the
// counts: 64 lists of 2000, V = 128256 14.1 / - / 10.1 us, of 8000 21.7 / 25.2 / 14.3, of 20000 45.9 / 53.3 / 25.2; 130 of 8000, V = 152064 28.0 / 43.7 / 23.1; 24 of 5000, V = 50000 16.1 / 15.1 / 11.7.
// Walked over bits: up to 1.06 below 500 ids, at most 1.00 from 800 on.
// What the head works from (u.head_*, kept where union_feeds says so): the split, or nothing shared and every list whole, by how many pairs the shared ids cover in
// all sequences together; every workgroup comes to the same answer from the counts.
template <int N>
__global__ __launch_bounds__(kListThreads) void union_lists_kernel(VocabPtrs p, UnionPtrs u, int batch, int groups, int tables) {
  constexpr int NW = kListThreads / 64;
  static_assert(NW == 16, "a row of lanes holds one total per wavefront");
  extern __shared__ __attribute__((aligned(16))) uint4 tab[];   // per word: shared bits, active shared bits, rank of the first shared bit, active shared bits before
  __shared__ int s_shared[NW], s_active[NW], s_rest[NW], s_pairs[NW], s_cover[NW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, b = blockIdx.x, w0 = tid * N;
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
  int2 part = make_int2(0, 0);
  if (u.parts && tid < (p.nwords + 15) / 16) part = u.parts[tid];        // at most 1024 of them: a state has fewer than 16384 words
  for (int i = tid; i < u.shared_cap; i += kListThreads) mypos[i] = -1;   // shared ids the sequence lacks, and room that none takes; the barriers below are between these and the columns
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
    const int pi = wave_incl_scan(part.x), ci = wave_incl_scan(part.y);
    if (lane == 63) {
      s_pairs[wave] = pi;
      s_cover[wave] = ci;
    }
  }
  __syncthreads();
  const int ts = s_shared[lane & 15], ta = s_active[lane & 15];
  int r = row_sum((lane & 15) < wave ? ts : 0) + si - ns;                // rank of this thread's first shared bit
  int pos = row_sum((lane & 15) < wave ? ta : 0) + ai - na;              // column of its first active bit
  const int all = row_sum(ts), listed = all < u.shared_cap ? all : u.shared_cap;
  bool split = false;
  if (u.parts) {
    const int pairs = row_sum(s_pairs[lane & 15]);
    split = union_split_pairs(pairs, pairs - row_sum(s_cover[lane & 15]));
  }
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
  const int tr = s_rest[lane & 15], nrest = row_sum(tr);
  int q = row_sum((lane & 15) < wave ? tr : 0) + ri - nr;
  int32_t* rid = u.rest_ids + (size_t)b * p.cap;
  int32_t* rpos = u.rest_pos + (size_t)b * p.cap;
  int32_t* hid = u.parts ? u.head_ids + (size_t)b * p.cap : nullptr;
  int32_t* hpos = u.parts ? u.head_pos + (size_t)b * p.cap : nullptr;
  if ((tid * batch) >> 10 == b) {                                        // this workgroup's share of the list of shared ids
    int at = r;
#pragma unroll
    for (int i = 0; i < N; ++i)
      for (uint32_t x = sh[i]; x; x &= x - 1u) u.shared_ids[at++] = (w0 + i) * 32 + __ffs(x) - 1;
  }
  if (tables && n > kWalkFrom) {
    int rank = r, before = pos - q;                                      // active shared bits before this thread's words
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (w0 + i < p.nwords) tab[w0 + i] = make_uint4(sh[i], ac[i] & sh[i], (uint32_t)rank, (uint32_t)before);
      rank += __popc(sh[i]);
      before += __popc(ac[i] & sh[i]);
    }
    __syncthreads();
    const int32_t* ids = p.ids + (size_t)b * p.cap;
    for (int j = tid; j < n; j += kListThreads) {
      const int id = ids[j];
      const uint4 t = tab[id >> 5];
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
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      for (uint32_t x = ac[i]; x; x &= x - 1u) {
        const uint32_t bit = x & (0u - x);
        const int id = (w0 + i) * 32 + __ffs(x) - 1;
        if (sh[i] & bit) {
          mypos[r + __popc(sh[i] & (bit - 1u))] = pos;
        } else {
          rid[q] = id;
          rpos[q] = pos;
          if (hid && split) {
            hid[q] = id;
            hpos[q] = pos;
          }
          ++q;
        }
        if (hid && !split) {
          hid[pos] = id;
          hpos[pos] = pos;
        }
        ++pos;
      }
      r += __popc(sh[i]);
    }
  }
  if (b == 0)
    for (int g = tid; g < groups; g += kListThreads) {
      u.shared_n[g] = listed;
      if (hid) u.head_shared_n[g] = split ? listed : 0;
    }
  if (tid == 0) {
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
  if (st->un.parts) union_count_kernel<true><<<(nw + 15) / 16, 1024, 0, s>>>(st->vp, st->un, st->batch);
  else union_count_kernel<false><<<(nw + 15) / 16, 1024, 0, s>>>(st->vp, st->un, st->batch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t tables = 16ll * nw;                                       // of lists that are walked; 300 000 ids and more are always written from the bits
  const int walk = st->vp.cap > kWalkFrom && tables <= kListsLds;
  const unsigned lds = walk ? (unsigned)tables : 0u;
  if (nw <= kListThreads) union_lists_kernel<1><<<st->batch, kListThreads, lds, s>>>(st->vp, st->un, st->batch, st->un_groups, walk);
  else if (nw <= 2 * kListThreads) union_lists_kernel<2><<<st->batch, kListThreads, lds, s>>>(st->vp, st->un, st->batch, st->un_groups, walk);
  else if (nw <= 4 * kListThreads) union_lists_kernel<4><<<st->batch, kListThreads, lds, s>>>(st->vp, st->un, st->batch, st->un_groups, walk);
  else if (nw <= 8 * kListThreads) union_lists_kernel<8><<<st->batch, kListThreads, lds, s>>>(st->vp, st->un, st->batch, st->un_groups, walk);
  else if (nw <= 16 * kListThreads) union_lists_kernel<16><<<st->batch, kListThreads, lds, s>>>(st->vp, st->un, st->batch, st->un_groups, walk);
  else return hipErrorInvalidValue;                                       // more ids than a state takes: its bitmaps fill LDS three times over
  return hipGetLastError();
}

}  // namespace nanospec
