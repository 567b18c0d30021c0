// The paper's own system design as a component (Sec. 3.3 "Avoiding sparse computation via asynchronous
// gathering"; the weight-gather row of Table 4; the repacked-weights row of Table 6): a pre-allocated packed
// buffer holds one copy of every active row; after a vocabulary update only the rows of ids that entered the
// active set are copied in -- on a stream of the caller's choice, so that the copy hides behind the draft
// backbone -- and the head is a dense product on the packed buffer.
//
// Slots are stable: an id keeps its slot while it stays active, a leaving id frees its slot, an entering id
// takes the lowest free one.  Slot order is therefore not id order; the head kernels write the logits of the row
// in slot s to the column out_pos[s] = position of that id in the ascending active list, so logits come out in
// exactly the layout of nanospec_sparse_head and the selection (ties by lower id) applies unchanged.
#include "common.h"

namespace nanospec {

constexpr int kSyncThreads = 1024;

// exclusive rank of `pred` among the workgroup's threads in thread order, and the workgroup total; sc: 17 ints of LDS
__device__ __forceinline__ int block_rank(bool pred, int* sc, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long bal = __ballot(pred);
  const int before = __popcll(bal & ((1ull << lane) - 1ull));
  __syncthreads();                                   // sc may still be read from the previous call
  if (lane == 0) sc[wave] = __popcll(bal);
  __syncthreads();
  int off = 0, tot = 0;
  for (int w = 0; w < kSyncThreads / 64; ++w) {
    const int t = sc[w];
    off += w < wave ? t : 0;
    tot += t;
  }
  *total = tot;
  return off + before;
}

// One workgroup: bring slot tables in line with the active list of sequence 0.
//   1. every slot whose id is no longer active (window bitmap | T bitmap) is freed;
//   2. the free slots are listed in ascending order;
//   3. every active id without a slot takes the next free one and goes on the copy list;
//   4. out_pos[slot] = position of the slot's id in the ascending list; hi = slots that may hold a row.
__global__ __launch_bounds__(kSyncThreads) void packed_sync_kernel(VocabPtrs p, PackedPtrs k) {
  __shared__ int sc[32];
  const int tid = threadIdx.x;
  const int n = p.n[0], cap = k.cap;
  int nfree = 0;
  for (int s0 = 0; s0 < cap; s0 += kSyncThreads) {
    const int s = s0 + tid;
    bool isfree = false;
    if (s < cap) {
      const int id = k.slot_id[s];
      isfree = id < 0;
      if (id >= 0) {
        const uint32_t bits = p.wbit[id >> 5] | p.tbit[id >> 5];
        if (!((bits >> (id & 31)) & 1u)) {
          k.slot_of[id] = -1;
          k.slot_id[s] = -1;
          k.out_pos[s] = -1;
          isfree = true;
        }
      }
    }
    int tot;
    const int r = block_rank(isfree, sc, &tot);
    if (isfree) k.free_list[nfree + r] = s;
    nfree += tot;
  }
  __syncthreads();                                   // free_list and slot_of are complete (one workgroup, one L1)
  int ncopy = 0, top = -1;
  for (int j0 = 0; j0 < n; j0 += kSyncThreads) {
    const int j = j0 + tid;
    int id = -1, sl = -1;
    if (j < n) {
      id = p.ids[j];
      sl = k.slot_of[id];
    }
    const bool fresh = j < n && sl < 0;
    int tot;
    const int r = block_rank(fresh, sc, &tot);
    if (fresh) {
      sl = k.free_list[ncopy + r];                   // n <= cap and every active id holds one slot: there is one
      k.slot_of[id] = sl;
      k.slot_id[sl] = id;
      k.copy_list[2 * (ncopy + r)] = id;
      k.copy_list[2 * (ncopy + r) + 1] = sl;
    }
    if (j < n) k.out_pos[sl] = j;
    top = max(top, sl);
    ncopy += tot;
  }
  // highest slot in use
  for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o));
  __syncthreads();
  if ((tid & 63) == 0) sc[tid >> 6] = top;
  __syncthreads();
  if (tid == 0) {
    int t = -1;
    for (int w = 0; w < kSyncThreads / 64; ++w) t = max(t, sc[w]);
    k.scal[0] = t + 1;                               // hi
    k.scal[1] = ncopy;
  }
}

// The same for capacities of up to Q x 4096 slots in one memory round trip.  What bounds it is instruction issue on its one compute unit and the address
// rate of scattered look-ups, a cycle per lane: every slot's id in both bitmaps and every listed id's slot were 12 of them per thread.  Here the bitmaps come into LDS in whole
// lines; a kept slot's position in the list is the rank of its id in the bitmap (words before it, from one scan, and bits below it), and the ids that enter are the
// active bits that no slot holds.  Thread t holds slots q * 4096 + 4t .. + 3 and wpt consecutive bitmap words.  The f-th free slot is taken by the f-th entering id, both
// ascending; the thread that holds a slot clears its tables only if it stays free.  No table by id is kept.  With the copy's launch behind it, against the look-ups: 3776 slots
// 7.3 -> 4.9 us, 1280 6.0 -> 4.8, 8000 10.2 -> 6.2, 15936 (then a walk in 1024s) 18.3 -> 10.0; with scans over __shfl and one LDS read per total 7.35 us at 3776.
// Sixteen wavefronts share four SIMDs, so an instruction that all execute costs 7 ns: scans are DPP chains, two counts of up to 16384 to a register.
template <int Q>
__global__ __launch_bounds__(kSyncThreads) void packed_sync_short_kernel(VocabPtrs p, PackedPtrs k) {
  constexpr int NW = kSyncThreads / 64, S = (Q + 1) / 2 + (Q > 1 ? 1 : 0);   // scans: (bits, free of q = 0), then two q each
  static_assert(NW == 16, "a row of lanes holds one total per wavefront");
  extern __shared__ __attribute__((aligned(16))) uint32_t smem[];   // active bits, bits that a slot holds, rank of each word's first bit; free slots
  uint32_t *act = smem, *held = smem + p.nwords;
  int *pre = reinterpret_cast<int*>(held + p.nwords), *s_free = pre + p.nwords;
  __shared__ int s_tot[S][NW], s_new[NW], s_top[NW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, cap = k.cap;   // a multiple of 64
  const int wpt = ((p.nwords + kSyncThreads - 1) / kSyncThreads + 3) & ~3;   // nwords is a multiple of 4
  const int w0 = tid * wpt, w1 = w0 + wpt < p.nwords ? w0 + wpt : p.nwords;
  int sid[Q][4];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int s = q * 4096 + tid * 4;
    const int4 a = *reinterpret_cast<const int4*>(k.slot_id + (s < cap ? s : 0));
    sid[q][0] = a.x; sid[q][1] = a.y; sid[q][2] = a.z; sid[q][3] = a.w;
  }
  int pop = 0;
  for (int w = w0; w < w1; w += 4) {
    const uint4 a = *reinterpret_cast<const uint4*>(p.wbit + w), t = *reinterpret_cast<const uint4*>(p.tbit + w);
    const uint4 v = make_uint4(a.x | t.x, a.y | t.y, a.z | t.z, a.w | t.w);
    *reinterpret_cast<uint4*>(act + w) = v;
    *reinterpret_cast<uint4*>(held + w) = make_uint4(0u, 0u, 0u, 0u);
    pop += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
  }
  __syncthreads();
  uint32_t fr[Q], gone[Q], word[Q][4];                     // bit e: slot free / by this call; the bitmap word of its id
  int top = -1;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    fr[q] = gone[q] = 0u;
    int mine = -1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // flags by arithmetic: with the two cases as branches the compiler lost the free bit of one of them (q = 1, e = 0)
      const int s = q * 4096 + tid * 4 + e, id = sid[q][e];
      word[q][e] = act[id >= 0 ? id >> 5 : 0];
      const uint32_t in = s < cap ? 1u : 0u, has = id >= 0 ? in : 0u, stays = has & (word[q][e] >> (id & 31));
      if (stays) atomicOr(&held[id >> 5], 1u << (id & 31));
      mine = stays ? s : mine;
      fr[q] |= (in & ~stays) << e;
      gone[q] |= (has & ~stays) << e;
    }
    const unsigned long long any = __ballot(mine >= 0);    // slots ascend with the lane
    if (any) top = __builtin_amdgcn_readlane(mine, 63 - __clzll((long long)any));
  }
  int incl[S];
  incl[0] = wave_incl_scan(pop << 16 | __popc(fr[0]));
#pragma unroll
  for (int i = 1; i < S; ++i) incl[i] = wave_incl_scan((2 * i < Q ? __popc(fr[2 * i < Q ? 2 * i : 0]) << 16 : 0) | __popc(fr[2 * i - 1]));
  if (lane == 63) {
#pragma unroll
    for (int i = 0; i < S; ++i) s_tot[i][wave] = incl[i];
    s_top[wave] = top;
  }
  __syncthreads();
  int before[S], total[S];
#pragma unroll
  for (int i = 0; i < S; ++i) {
    const int t = s_tot[i][lane & 15];
    before[i] = row_sum((lane & 15) < wave ? t : 0);
    total[i] = row_sum(t);
  }
  int fresh = 0, rank = (before[0] >> 16) + (incl[0] >> 16) - pop;
  for (int w = w0; w < w1; w += 4) {
    const uint4 v = *reinterpret_cast<const uint4*>(act + w), h = *reinterpret_cast<const uint4*>(held + w);
    int4 r;
    r.x = rank;
    r.y = r.x + __popc(v.x);
    r.z = r.y + __popc(v.y);
    r.w = r.z + __popc(v.z);
    rank = r.w + __popc(v.w);
    *reinterpret_cast<int4*>(pre + w) = r;
    fresh += __popc(v.x & ~h.x) + __popc(v.y & ~h.y) + __popc(v.z & ~h.z) + __popc(v.w & ~h.w);
  }
  const int ninc = wave_incl_scan(fresh);
  if (lane == 63) s_new[wave] = ninc;
  int fbase[Q], ftot = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i = (q + 1) / 2, sh = q > 0 && q % 2 == 0 ? 16 : 0, mask = 0xffff;
    fbase[q] = ftot + ((before[i] >> sh) & mask) + ((incl[i] >> sh) & mask) - __popc(fr[q]);
    ftot += (total[i] >> sh) & mask;
    int f = fbase[q];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if ((fr[q] >> e) & 1u) s_free[f++] = q * 4096 + tid * 4 + e;
  }
  __syncthreads();
  const int tn = s_new[lane & 15], ncopy = row_sum(tn);
  int r = row_sum((lane & 15) < wave ? tn : 0) + ninc - fresh;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int s = q * 4096 + tid * 4;
    int out[4], f = fbase[q];
    uint32_t taken = 0u;                                   // bit e: free slot that an entering id takes, which writes its tables
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int id = sid[q][e];
      const uint32_t isfree = (fr[q] >> e) & 1u;
      const int at = pre[id >= 0 ? id >> 5 : 0] + __popc(word[q][e] & ((1u << (id & 31)) - 1u));
      out[e] = isfree ? -1 : at;
      taken |= (f < ncopy ? isfree : 0u) << e;
      f += isfree;
    }
    if (s < cap) {
      if (taken == 0u) {
        *reinterpret_cast<int4*>(k.out_pos + s) = make_int4(out[0], out[1], out[2], out[3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!((taken >> e) & 1u)) k.out_pos[s + e] = out[e];
      }
      const uint32_t clear = gone[q] & ~taken;
      if (clear) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((clear >> e) & 1u) k.slot_id[s + e] = -1;
      }
    }
  }
  if (fresh)
    for (int w = w0; w < w1; ++w) {
      const uint32_t bits = act[w];
      for (uint32_t nb = bits & ~held[w]; nb; nb &= nb - 1u, ++r) {
        const int e = __ffs(nb) - 1, id = w * 32 + e, sl = s_free[r];   // n <= cap and every active id holds one slot: there is one
        k.slot_id[sl] = id;
        k.out_pos[sl] = pre[w] + __popc(bits & ((1u << e) - 1u));
        k.copy_list[2 * r] = id;
        k.copy_list[2 * r + 1] = sl;
      }
    }
  if (tid == 0) {
    int hi = ncopy > 0 ? s_free[ncopy - 1] : -1;           // free slots are taken in ascending order
#pragma unroll
    for (int w = 0; w < NW; ++w) hi = max(hi, s_top[w]);
    k.scal[0] = hi + 1;
    k.scal[1] = ncopy;
  }
}

// dynamic LDS of packed_sync_short_kernel; packed_sync_kernel where it is more than a compute unit has
constexpr int kSyncLds = 156 * 1024;
static int64_t sync_lds(const nanospec_state* st) { return 12ll * st->vp.nwords + 4ll * st->pk.cap; }

hipError_t packed_configure_device() {
  const void* fns[] = {reinterpret_cast<const void*>(packed_sync_short_kernel<1>), reinterpret_cast<const void*>(packed_sync_short_kernel<2>),
                       reinterpret_cast<const void*>(packed_sync_short_kernel<4>)};
  for (const void* f : fns) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kSyncLds);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Copy the listed rows W[id] -> buf[slot]: the weight-gather kernel.  Two small workgroups per compute unit (a decoding step copies a
// row or two, and then the launch is all there is: a request of 16 steps 365 us with 256 workgroups of 1024 threads, 359 with 512 of
// 256, 364 with 256 of 256), four 16-byte pieces per thread in flight for the first gather.
__global__ __launch_bounds__(256) void packed_copy_kernel(const uint4* __restrict__ W, PackedPtrs k, int row_vec /* 16-byte pieces per row */) {
  const int ncopy = k.scal[1];
  uint4* buf = reinterpret_cast<uint4*>(k.buf);
  const int64_t total = (int64_t)ncopy * row_vec, stride = (int64_t)gridDim.x * 256;
  for (int64_t t0 = (int64_t)blockIdx.x * 256 + threadIdx.x; t0 < total; t0 += 4 * stride) {
    uint4 v[4];
    int64_t to[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t t = t0 + u * stride;
      const uint32_t tc = (uint32_t)(t < total ? t : t0);   // below 2^32: capacity * d / 8
      const uint32_t e = tc / (uint32_t)row_vec, i = tc % (uint32_t)row_vec;
      const int2 cs = *reinterpret_cast<const int2*>(k.copy_list + 2 * (int64_t)e);
      v[u] = W[(int64_t)cs.x * row_vec + i];
      to[u] = (int64_t)cs.y * row_vec + i;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (t0 + u * stride < total) buf[to[u]] = v[u];
  }
}

__global__ __launch_bounds__(256) void packed_reset_kernel(PackedPtrs k, int V) {
  const int i = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
  for (int v = i; v < V; v += stride) k.slot_of[v] = -1;
  for (int s = i; s < k.cap; s += stride) {
    k.slot_id[s] = -1;
    k.out_pos[s] = -1;
  }
  if (i == 0) {
    k.scal[0] = 0;
    k.scal[1] = 0;
  }
}

hipError_t launch_packed_reset(const nanospec_state* st, hipStream_t s) {
  packed_reset_kernel<<<256, 256, 0, s>>>(st->pk, st->V);
  return hipGetLastError();
}

hipError_t launch_packed_gather(const nanospec_state* st, const void* W, hipStream_t s) {
  const int cap = st->pk.cap;
  const int64_t lds = sync_lds(st);
  if (cap > 16384 || lds > kSyncLds) packed_sync_kernel<<<1, kSyncThreads, 0, s>>>(st->vp, st->pk);
  else if (cap <= 4096) packed_sync_short_kernel<1><<<1, kSyncThreads, lds, s>>>(st->vp, st->pk);
  else if (cap <= 8192) packed_sync_short_kernel<2><<<1, kSyncThreads, lds, s>>>(st->vp, st->pk);
  else packed_sync_short_kernel<4><<<1, kSyncThreads, lds, s>>>(st->vp, st->pk);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  packed_copy_kernel<<<512, 256, 0, s>>>(static_cast<const uint4*>(W), st->pk, st->d / 8);
  return hipGetLastError();
}

}  // namespace nanospec
